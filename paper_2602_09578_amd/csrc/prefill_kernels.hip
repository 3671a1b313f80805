// Prefill (prompt) attention over the paged KV cache, and the scatter that puts a prompt's
// keys and values into its pages.  This is the step that creates, once per prompt, the prefix
// every sample of that prompt then shares (Parallel Sampling, Section 5.1 of the paper); the
// paper leaves the computation to its inference backend, so the operation is the textbook
// causal attention stated in marl_decode.h:
//   query token at position t of group g attends to positions 0..t of the group's pages.
// A group may bring only a chunk of its prompt (positions pos0 .. pos0+n-1): the earlier
// positions are then context that is already in the cache (chunked prefill).
//
// Structure.  Query rows of a (group, KV head) are flattened as rho = token * R + head-in-group
// and cut into equal blocks of at most kQB = 192 rows; one work item = (group, row block, KV
// head).  The item streams keys/values 0 .. (last position of the block) through a ring of four
// LDS step buffers, 32 tokens (two pages, 16 KB) per step, in the XOR-swizzled layout of the
// decode prefix kernel; the four waves split the block's 16-row tiles (up to three each).  The
// steps go from global memory straight into LDS (global_load_lds_dwordx4, no staging
// registers), which is what leaves room for the third tile: every wave reads the whole step out
// of LDS for its rows, so more rows per wave make the same reads do more work.  Causality
// costs little: a block spans kQB / R consecutive tokens, so only its last one or two steps need
// the per-row mask, and a tile skips steps that lie entirely beyond its rows.  A block that is
// taken whole sees all of its keys, so its output is normalised and written directly.
//
// Small calls are one launch (prefill_small_kernel): a workgroup per item, which it finds in the groups by itself.  The others:
// Work distribution: a one-workgroup plan kernel lists the row blocks group after group, inside a
// group last-first (most keys first), so that blocks of a group run at the same time and its keys come
// out of the caches; a list of at most kPfSorted blocks, but more items than workgroups, is put into falling order of cost instead
// (so few items end evenly only if the long ones start first: 494 blocks x 4 heads of 47 short prompts
// would take 1.20 times their even share, sorted 1.04).  Item i = (block i / Hkv, KV head i % Hkv).  A
// workgroup starts with item b and knows its next item while it works on one: that item's steps follow
// the current one's in the ring without a gap, and its queries are requested before the current rows
// are written.  The second item is fixed, every further one is drawn from a counter when the one before
// the one before it ends.  (A fixed assignment instead of the counter left 3 to 13 % of the time to the
// longest share; items drawn another item earlier left the ends of short lists uneven.)
//   A few long items (chunks of a few prompts behind long context) leave workgroups idle, or end unevenly,
// whatever their order.  For a sorted list the plan kernel therefore weighs dividing long blocks along their
// keys: a part's sums (float32, unnormalised) go to the workspace, and the workgroup that arrives last at a
// block adds the parts.  Whole and divided: one chunk of 512 tokens behind 8192, 64 / 8 heads 215 -> 175 us,
// 28 / 4 heads 253 -> 94 us; 64 tokens behind 2000, 64 / 8 heads, 70 -> 40 us; one prompt of 2048 tokens, 28 / 4 heads,
// 79 -> 66 us; six chunks of up to 512 behind up to 8192, 64 / 8 heads, 382 -> 357 us.  Lists with more work than that
// stay whole (9 chunks of 512 behind up to 8000, 591 and 584 us), and run the code without parts (22 spilled
// scalar registers instead of 86; 2 to 3 % of such a list's time).
// A workspace with room for the list alone is served with whole blocks.
//
// What bounds it: the issue of instructions at the clock that its power leaves (1.81 GHz on the 256 prompts below).  A step of a
// wave is 48 matrix instructions (768 cycles
// of the matrix core) and about 100 vector instructions, 24 of them exponentials (710 cycles of the
// vector ALU), and the two waves of a SIMD overlap little of it: 1.58 us per step and workgroup at
// two workgroups per CU with 141 vector and 105 scalar instructions, 1.37 with 120 and 50 (page
// ids and addresses of the loads, LDS addresses, no test of the eight scores' maximum).  The same step alone, over and over on LDS data
// and without items, runs at 1.43 PFLOP/s, with loads that the caches hold at 1.28.  256 prompts of
// 512 to 2048 tokens, 28 / 4 heads: 3.99 -> 3.52 ms (0.98 PFLOP/s; a large matrix product of this
// card: 1.19); six chunks behind up to 8192 tokens, 64 / 8 heads: 0.43 -> 0.37 ms.  An item takes about 6 us beside its
// steps (rows written 2.6, the next item read and queries requested 2.2, two steps on the causal edge 0.6), in which the
// other workgroup of the CU has it alone; 7.5 with output rows through LDS, a first step taken twice
// and maxima in every step on the edge (46 prompts of up to 1666, 28 / 4 heads: 604 -> 586 us; 33 of up to 2730, 4 / 4 heads: 148 -> 143).
// Memory costs clock, not cycles: with an item
// bound ahead a prompt's blocks run further apart in time than one after the other did, and the 256 prompts fetch
// 15 GB instead of 8.2; with all groups on the pages of one prompt, which the caches hold, they fetch 5.5 GB, take as many cycles
// (6.59 M) and 5 % less time (3.63 and 3.44 ms on one card): what the traffic takes is power, and with it 0.1 GHz.
#include <algorithm>

#include "marl_internal.h"
#include "wave_ops.h"

namespace marl {
namespace {

#ifndef MARL_PREFILL_MT
#define MARL_PREFILL_MT 3
#endif
#ifndef MARL_PREFILL_NW
#define MARL_PREFILL_NW 4
#endif
#ifndef MARL_PREFILL_WAVES_PER_EU
#define MARL_PREFILL_WAVES_PER_EU 2
#endif
constexpr int kMT = MARL_PREFILL_MT;          // 16-row tiles per wave
constexpr int kNW = MARL_PREFILL_NW;          // waves per workgroup
constexpr int kQB = 16 * kMT * kNW;           // most query rows of one work item
constexpr int kPfThreads = 64 * kNW;
constexpr int kPfStepBytes = 2 * kBlockTok * kD * 2;   // K + V of one 32-token step
constexpr int kPlanThreadsPf = 1024;

// LDS step buffers, filled by direct global-to-LDS loads (two workgroups of at most 80 KB per CU)
constexpr int kPfStages = 4;
struct PrefillLds {
  __attribute__((aligned(16))) char buf[kPfStages][kPfStepBytes];
  int arrived;   // parts of the current block that were finished before this one
  int next;      // a drawn item
  int late;      // an item drawn when nothing was left to do
};
// s_waitcnt immediate that waits only for the vector-memory counter to drop to n (gfx9 encoding)
constexpr int pf_lgkmcnt0 = 0xf | (3 << 14) | (7 << 4);   // waits only for LDS and scalar operations
constexpr int pf_vmcnt_imm(int n) { return (n & 0xf) | ((n >> 4) << 14) | (7 << 4) | (0xf << 8); }

// counters at the head of the workspace (same slots as the decode plan uses, so that
// marl_attn_read_flags reads this workspace too); the header is followed by num_groups + 1 words, of which the last is
// the length of the list
constexpr int kPfCursor = MARL_CTR_PREFIX_CURSOR, kPfFlags = MARL_CTR_FLAGS;
constexpr int kPfLate = 17;      // items that were drawn late
constexpr int kPfIsSorted = 18;  // not zero: the list is in falling order of cost
constexpr int kPfDivided = 16;   // not zero: the list holds parts of blocks (a word that the decode plan does not use)

// n_g usable query tokens of group g (clamped to the q array and to the table row)
__device__ __forceinline__ int group_tokens(const PrefillArgs& a, int g, int& flag) {
  const int b = a.q_start[g], e = a.q_start[g + 1], p0 = a.q_pos0[g];
  int n = e - b;
  if (b < 0 || e > a.NT || n < 0 || p0 < 0) { flag |= MARL_FLAG_BAD_GROUP; return 0; }
  const long room = (long)a.max_pp * kPage - p0;
  if (n > room) { flag |= MARL_FLAG_LEN_CLAMPED; n = room > 0 ? (int)room : 0; }
  return n;
}

// A group's nrows query rows are cut into ceil(nrows / kQB) blocks of equal size (a multiple of
// 16 rows), not into full blocks and a remainder: 224 rows are two blocks of 112 (7 tiles each
// over the waves), not 192 + 32.
__device__ __forceinline__ int blocks_of(int nrows) { return (int)(((uint32_t)nrows + kQB - 1) / kQB); }
__device__ __forceinline__ int block_rows(int nrows, int nb) {
  return (int)((((uint32_t)nrows + nb - 1) / (uint32_t)nb + 15) / 16 * 16);
}

// A list record: the group and the block's first row (a multiple of 16) with the number of 16-row
// tiles of the group's blocks in the low four bits.
static_assert(kQB / 16 < 16, "a block's tiles are packed into four bits");
__device__ __forceinline__ int2 pack_item(int g, int row_begin, int qb) { return make_int2(g, row_begin | (qb >> 4)); }

constexpr int kPfSorted = 512;    // a list of at most so many entries is sorted
constexpr int kPfClasses = 64;    // cost classes of that order
constexpr int kPfMaxDiv = 16;     // most parts of one block's keys (four bits of a list record)
constexpr int kPfLongKeys = 960;  // keys: a list of shorter blocks stays whole (820 keys each, 228 items: 38 us, divided 47; 1000 keys: 43.8 and 42)
constexpr int kPfMinPart = 512;   // keys: no part is meant to be shorter
// lengths of parts that are considered, in even shares of a workgroup
__constant__ constexpr float kPfLens[16] = {0.f, 0.5f, 0.625f, 0.75f, 0.875f, 1.f, 1.125f, 1.25f, 1.5f, 1.75f, 2.f, 2.5f, 3.f, 4.f, 6.f, 8.f};
constexpr int kPfSplitBit = (int)0x80000000u;   // in a record's group: the entry is one part of the block's keys

// What bounds it: the chain of its one workgroup's barriers and LDS round trips, and the stores of the list.  A group per
// thread wrote hundreds of blocks one after the other, and one wave sorted a list and wrote its parts: now a wave writes a long
// group, and eight waves have an entry per thread.  (16 prompts of up to 3798 tokens, 16 / 1 heads, 5000 blocks: 61.4 us,
// now 5.6; 6 of up to 3132, 64 / 8 heads: 22.6, now 5.2; 3 of up to 1635, 28 / 4, weighed and in parts: 15.6, now 8.5;
// 13 of up to 46, 28 / 4: 4.3, now 4.0.)
__global__ __launch_bounds__(kPlanThreadsPf) void prefill_plan_kernel(PrefillArgs a) {
  constexpr int kWavesPf = kPlanThreadsPf / 64;
  __shared__ long long wave_sum[kWavesPf];   // 64-bit: inconsistent inputs must not wrap the sums
  __shared__ int hist[kPfClasses], starts[kPfClasses];
  __shared__ int4 groups[kPlanThreadsPf];   // first entry, blocks, rows of a block, q_pos0
  __shared__ int2 list[kPfSorted];     // the first blocks and their groups' q_pos0: a short list never goes through memory
  __shared__ int list_pos0[kPfSorted];
  __shared__ int flags_all, end_all, parts_used, most_keys, fewest, most, entries_all;
  __shared__ float estimate[kWavesPf];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int flag = 0;
  if (tid == 0) {
    flags_all = end_all = parts_used = most_keys = most = entries_all = 0;
    fewest = 0x7fffffff;
  }
  if (tid < kPfClasses) hist[tid] = 0;
  __syncthreads();
  auto put = [&](int at, int2 rec, int pos0) {
    if (at < kPfSorted) {
      list[at] = rec;
      list_pos0[at] = pos0;
    } else {
      a.items[at] = rec;
    }
  };
  long long carry = 0;
  for (int g0 = 0; g0 < a.NG; g0 += kPlanThreadsPf) {
    const int g = g0 + tid;
    int nb = 0, nrows = 0, pos0 = 0;
    if (g < a.NG) {
      nrows = group_tokens(a, g, flag) * a.R;   // (at most all rows of q: less than 2^31)
      nb = blocks_of(nrows);
      pos0 = a.q_pos0[g];
    }
    // groups that overlap in q could ask for more blocks than the workspace was sized for
    // (its bound assumes they share no rows): such a group is dropped
    if (nb > a.max_blocks) { nb = 0; flag |= MARL_FLAG_BAD_GROUP; }
    const long long inc = wave_inclusive_scan((long long)nb);
    if (lane == 63) wave_sum[wave] = inc;
    const bool long_groups = __syncthreads_or(nb > 16);
    long long before = carry, all = 0;
#pragma unroll
    for (int w = 0; w < kWavesPf; ++w) {
      const long long v = wave_sum[w];
      before += w < wave ? v : 0;
      all += v;
    }
    int first = a.max_blocks;
    if (g < a.NG) {
      const long long first64 = before + inc - nb;
      if (first64 + nb > a.max_blocks) {   // as above; every later group then fails this test too
        flag |= MARL_FLAG_BAD_GROUP;
        nb = 0;
      } else {
        first = (int)first64;
        if (nb) {
          atomicMax(&end_all, first + nb);
          atomicMax(&most_keys, pos0 + nrows / a.R);
        }
      }
    }
    // the groups' blocks, last (most keys) first
    const int qb = nb ? block_rows(nrows, nb) : 0;
    if (!long_groups) {   // workgroup-uniform
      for (int k = 0; k < nb; ++k) put(first + k, pack_item(g, (nb - 1 - k) * qb, qb), pos0);
    } else {
      groups[tid] = make_int4(first, nb, qb, pos0);
      __syncthreads();
      for (int k0 = wave; k0 < min(kPlanThreadsPf, a.NG - g0); k0 += kWavesPf) {   // wave-uniform
        const int4 v = groups[k0];
        for (int k = lane; k < v.y; k += 64) put(v.x + k, pack_item(g0 + k0, (v.y - 1 - k) * v.z, v.z), v.w);
      }
    }
    carry += all;
    __syncthreads();
  }
  if (flag) atomicOr(&flags_all, flag);
  __syncthreads();
  // The accepted groups' blocks are exactly [0, end_all).
  int total = end_all;   // (then entries of the list)
  const int blocks = total;
  // A list of at most one item per workgroup needs no order; blocks of up to kPfLongKeys keys are not divided.
  const bool weigh = total <= kPfSorted && a.split_slots > 0 && most_keys > kPfLongKeys;
  const bool sorted = total <= kPfSorted && (weigh || (long)total * a.Hkv > a.slots);
  if (!sorted)
    for (int k = tid; k < min(total, kPfSorted); k += kPlanThreadsPf) a.items[k] = list[k];
  // keys of a block: what its rows see, rounded up to whole rows of it
  auto keys_of = [&](int k) { return list_pos0[k] + ((list[k].y & ~15) + (list[k].y & 15) * 16) / a.R; };
  float part_len = 0.f;   // keys that a part has at most; 0: whole blocks
  auto parts_of = [&](int keys, float len) { return len > 0.f && keys > 0 ? min(kPfMaxDiv, (int)ceilf((float)keys / len)) : 1; };
  if (weigh) {
    for (int k = tid; k < kPfMaxParts; k += kPlanThreadsPf) a.split_arrived[k] = 0;
    // Every wave holds the list's blocks.
    constexpr int kPer = kPfSorted / 64;
    int keys[kPer];
    float all = 0.f;
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      keys[u] = -1;
      if (u * 64 < blocks) keys[u] = u * 64 + lane < blocks ? keys_of(u * 64 + lane) : -1;
      all += (float)max(keys[u], 0);
    }
    // Wave w estimates the time, in keys, with blocks divided into parts of at most kPfLens[w] even shares
    // (wave 0: whole blocks): the longest item if all run at once, else an even share of
    // all items and half an item.  An item costs 128 keys beside its own, a part more, and a part's sums are
    // written and read back in everybody's time (200 KB at 4 TB/s): 400 and 0.9 keys, or, in lists that take several
    // rounds also whole, whose other items run meanwhile, 228 and 0.4.  Checked on 434 drawn shapes that none
    // of this was chosen by (1 to 64 chunks of up to 4096 tokens behind up to 8192), each timed with all of the sixteen
    // lengths: the time of the length that is taken is 1.5 % above the best one's in the geometric mean, whole
    // lists' is 26 %; 9 shapes are slower than whole by more than 2 %, the worst by 9 %.  The optimum is flat: 228 and
    // 1.1 in both kinds of list gave 1.5 % and 10 shapes, among others a prompt of 1172 tokens, 64 / 8 heads, 47.5 us
    // (whole 45.2), 60 of up to 78 behind up to 991, 16 / 1 heads, 49.5 (now 47.6).
    const bool rounds = (long)blocks * a.Hkv > a.split_slots;
    const float part_extra = rounds ? 228.f : 400.f, part_all = rounds ? 0.4f : 0.9f;
    auto sum_all = [](float v) { return wave_allreduce(v, [](float x, float y) { return x + y; }); };
    const float slots = (float)a.split_slots, share = sum_all(all) * (float)a.Hkv / slots;
    auto len_of = [&](int w) { return w > 0 ? fmaxf((float)kPfMinPart, kPfLens[w] * share) : 0.f; };
    const float len = len_of(wave);
    float items = 0.f, in_parts = 0.f, work = 0.f, longest = 0.f;
#pragma unroll
    for (int u = 0; u < kPer; ++u)
      if (keys[u] >= 0) {
        const int parts = parts_of(keys[u], len);
        const float n = (float)parts, extra = parts > 1 ? part_extra : 128.f;
        items += n;
        in_parts += parts > 1 ? n : 0.f;
        work += (float)keys[u] + n * extra;
        longest = fmaxf(longest, (float)keys[u] / n + extra);
      }
    const float entries = sum_all(items);
    items = entries * (float)a.Hkv;
    in_parts = sum_all(in_parts) * (float)a.Hkv;
    work = sum_all(work) * (float)a.Hkv;
    longest = wave_allreduce(longest, [](float x, float y) { return fmaxf(x, y); });
    const float time = (items <= slots ? longest : fmaxf(longest, work / slots + 0.5f * work / items)) + part_all * in_parts;
    // (no more than the list and the partial results have room for; whole blocks unless 3 % of such a list's time, else 7 %, are gained)
    const bool fits = entries <= (float)kPfSorted && in_parts <= (float)kPfMaxParts;
    if (lane == 0) estimate[wave] = wave == 0 ? (rounds ? 0.97f : 0.93f) * time : fits ? time : INFINITY;
    __syncthreads();
    const float mine = estimate[lane & (kWavesPf - 1)];
    const float least = wave_allreduce(mine, [](float x, float y) { return fminf(x, y); });
    part_len = len_of(__builtin_ctzll(__builtin_amdgcn_ballot_w64(mine == least)));   // (the first of the least)
  }
  if (sorted) {   // workgroup-uniform: a counting sort over kPfClasses classes between the fewest and the most keys
    const bool entry = tid < blocks;   // (at most kPfSorted)
    int keys = entry ? keys_of(tid) : 0;
    const int parts = entry ? parts_of(keys, part_len) : 0;
    if (entry) keys /= parts;
    if (wave < kPfSorted / 64) {
      const int lo = wave_allreduce(entry ? keys : 0x7fffffff, [](int x, int y) { return min(x, y); });
      const int hi = wave_allreduce(keys, [](int x, int y) { return max(x, y); });
      const int n = wave_allreduce(parts, [](int x, int y) { return x + y; });
      if (lane == 0) {
        atomicMin(&fewest, lo);
        atomicMax(&most, hi);
        atomicAdd(&entries_all, n);
      }
    }
    __syncthreads();
    const int width = max(1, (most - fewest) / kPfClasses + 1), cls = (most - keys) / width;
    if (entry) atomicAdd(&hist[cls], parts);
    __syncthreads();
    if (wave == 0) {
      const int c = hist[lane];
      starts[lane] = wave_inclusive_scan(c) - c;
    }
    __syncthreads();
    if (entry) {
      const int at = atomicAdd(&starts[cls], parts);
      const int2 rec = list[tid];
      if (parts == 1) {
        a.items[at] = rec;
      } else {
        const int first_part = atomicAdd(&parts_used, parts);
        for (int k = 0; k < parts; ++k) {
          a.items[at + k] = make_int2(rec.x | kPfSplitBit, rec.y);
          a.split_info[at + k] = (first_part << 8) | (k << 4) | (parts - 1);
        }
      }
    }
    __syncthreads();
    total = entries_all;
  }
  if (tid == 0) {
    *a.list_length = total;
    a.counters[kPfCursor] = 0;
    a.counters[kPfLate] = 0;
    a.counters[kPfIsSorted] = sorted;
    a.counters[kPfDivided] = parts_used;
    a.counters[kPfFlags] = flags_all;   // the attention kernel may add MARL_FLAG_BAD_PAGE
  }
}
static_assert(kPfClasses == 64, "one class per lane in the scan");

typedef const char __attribute__((address_space(1))) * GlobalBytes;
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
// Scalar load of element `at` of a wave-uniform array (scalar base + 32-bit offset).
__device__ __forceinline__ int ld_uniform_at(const int32_t* p, uint32_t at) {
  const char __attribute__((address_space(4))) * base =
      reinterpret_cast<const char __attribute__((address_space(4)))*>(reinterpret_cast<uintptr_t>(p));
  return *reinterpret_cast<const int32_t __attribute__((address_space(4)))*>(base + at * 4u);
}

// What one item is, wave-uniform (scalar registers).
struct PfItem {
  const int32_t* table_row;   // page ids of the group
  int kvh, rows;
  int tok0, rem0;             // the block's first row = tok0 * R + rem0
  int qrow0, pos0;            // row of q and position of token tok0
  int tok_end;                // keys the block needs: 0 .. position of its last row
  int step0, nsteps, slots;   // key steps step0 .. nsteps - 1; the slot of the ring behind its last (at least kPfStages after step0)
  int split;                  // -1: all of the block's keys; else first part << 8 | this part << 4 | parts - 1
};

// x / R for 0 <= x < 65536 / 16 with inv_R = ceil(65536 / R): exact, since x (inv_R R - 65536) < 65536
__device__ __forceinline__ int div_R(int x, int inv_R) { return (x * inv_R) >> 16; }

// A small call has no plan kernel: every workgroup goes over the groups, one per thread, until it has found its block in the
// plan's list (the groups' blocks in their order, last block of a group first), and the one that sets the flags over all of them.
//   visit(group, tokens, blocks, blocks up to this group's last): for every group that the plan would list (wave-uniform calls
//   are not promised), in rounds of kPfThreads groups, up to the one in which block `until` has gone by.
struct FindLds {
  int wave_blocks[kNW];
  int group, packed, flags;
};
template <class Visit>
__device__ __forceinline__ void walk_groups(const PrefillArgs& a, const int until, int& flag, FindLds& lds, Visit&& visit) {
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int before = 0;                      // blocks of the groups so far
  for (int g0 = 0; g0 < a.NG && before <= until; g0 += kPfThreads) {   // workgroup-uniform
    const int g = g0 + tid;
    int n = 0, nb = 0;
    if (g < a.NG) {
      n = group_tokens(a, g, flag);
      nb = blocks_of(n * a.R);
      if (nb > a.max_blocks) { nb = 0; flag |= MARL_FLAG_BAD_GROUP; }   // (dropped, as in the plan)
    }
    const int inc = wave_inclusive_scan(nb);
    __syncthreads();                   // (the waves' numbers of the round before have been read)
    if (lane == 63) lds.wave_blocks[wave] = inc;
    __syncthreads();
    int end = before + inc;
#pragma unroll
    for (int w = 0; w < kNW; ++w) {
      if (w < wave) end += lds.wave_blocks[w];
      before += lds.wave_blocks[w];
    }
    if (g < a.NG && end > a.max_blocks) flag |= MARL_FLAG_BAD_GROUP;   // (past the room for blocks: dropped, too)
    else if (nb > 0) visit(g, n, nb, end);
  }
}
__device__ __forceinline__ bool find_block(const PrefillArgs& a, const int block, int& g, int& packed, FindLds& lds) {
  if (threadIdx.x == 0) lds.group = -1;
  int flag = 0;
  walk_groups(a, block, flag, lds, [&](int group, int n, int nb, int end) {
    if (end > block && end - nb <= block) {
      const int qb = block_rows(n * a.R, nb);
      lds.group = group;
      lds.packed = pack_item(group, (end - 1 - block) * qb, qb).y;
    }
  });
  __syncthreads();
  g = __builtin_amdgcn_readfirstlane(lds.group);
  packed = __builtin_amdgcn_readfirstlane(lds.packed);
  return g >= 0;
}

template <bool kSplit>
__device__ __forceinline__ PfItem item_of(const PrefillArgs& a, const int block, const int kvh, const int g_rec, const int packed) {
  PfItem it;
  it.kvh = kvh;
  const int g = kSplit ? g_rec & ~kPfSplitBit : g_rec;
  const int b = ld_uniform(a.q_start + g), e = ld_uniform(a.q_start + g + 1);
  const int pos0 = ld_uniform(a.q_pos0 + g);
  const int row_begin = packed & ~15;
  // (a listed group passed the plan's checks; its tokens are clamped to the table row as there)
  const int nrows = (int)min((long)(e - b), (long)a.max_pp * kPage - pos0) * a.R;
  it.rows = min((packed & 15) * 16, nrows - row_begin);
  it.tok0 = row_begin / a.R;
  it.rem0 = row_begin - it.tok0 * a.R;
  it.qrow0 = b + it.tok0;
  it.pos0 = pos0 + it.tok0;
  it.tok_end = it.pos0 + div_R(it.rem0 + it.rows - 1, a.inv_R) + 1;
  it.nsteps = (it.tok_end + kBlockTok - 1) / kBlockTok;
  it.step0 = 0;
  it.split = -1;
  if (kSplit && g_rec < 0) {
    it.split = ld_uniform(a.split_info + block);
    const uint32_t k = (it.split >> 4) & 15, parts = (it.split & 15) + 1, all = it.nsteps;
    it.step0 = (int)(all * k / parts);
    it.nsteps = (int)(all * (k + 1) / parts);
  }
  it.slots = max(it.nsteps, it.step0 + kPfStages);
  it.table_row = a.prefix_table + (size_t)g * a.max_pp;
  return it;
}

template <bool kSplit>
__device__ __forceinline__ PfItem read_item(const PrefillArgs& a, int qi) {
  const int block = qi / a.Hkv;
  const int32_t* rec = reinterpret_cast<const int32_t*>(a.items + block);
  const int g_rec = ld_uniform(rec), packed = ld_uniform(rec + 1);
  return item_of<kSplit>(a, block, qi - block * a.Hkv, g_rec, packed);
}

// Items of one workgroup, one after the other: first(), `second` and the drawn ones, as far as they are less than n_ahead
// (kAlone: only first()).
template <bool kSplit, bool kAlone, class First>
__device__ __forceinline__ void prefill_items(const PrefillArgs& a, First&& first, const int second, const int n_ahead,
                                              PrefillLds& lds, int& bad_page) {
  constexpr int kLoads = 1024 / (kNW * 64);     // 16-byte loads per thread and step (16 KB per step)
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int i = lane & 15, j = lane >> 4;
  const float sc = fmaxf(fabsf(a.scale) * 1.44269504088896340736f, 1e-30f);
  const uint32_t sign_flip = a.scale < 0.f ? 0x80008000u : 0u;
  // this wave's tiles: wave, wave + kNW, ...; tile_lo / tile_hi: fewest / most keys any of its rows sees
  // (per-lane row data is computed where it is used, from a lane number the compiler cannot see
  // through: kept, it would take registers through the loops that they do not have)
  int tile_lo[kMT], tile_hi[kMT];
  auto opaque_lane = [&] { int l = lane; asm volatile("" : "+v"(l)); return l; };
  // this lane's row of a tile: its index in q and out (-1: none) and the number of keys it sees
  auto row_at = [&](const PfItem& it, int r, int& tok) {
    const int rho = it.rem0 + r;
    tok = div_R(rho, a.inv_R);   // from the block's first token on
    return (it.qrow0 + tok) * a.Hq + it.kvh * a.R + (rho - tok * a.R);
  };
  auto row_of = [&](const PfItem& it, int qt, int row16, int& sees) {
    const int r = (qt * kNW + wave) * 16 + row16;
    int tok;
    const int idx = row_at(it, r, tok);
    sees = r < it.rows ? it.pos0 + tok + 1 : 1;
    return r < it.rows ? idx : -1;
  };
  u32x4 qreg[kMT][4];
  auto load_rows = [&](const PfItem& it) {
    const int l = opaque_lane();
#pragma unroll
    for (int qt = 0; qt < kMT; ++qt) {
      const int r0 = (qt * kNW + wave) * 16;            // first row of the tile within the block
      tile_lo[qt] = tile_hi[qt] = 0;                    // tile without rows: never computed
      if (r0 < it.rows) {
        tile_lo[qt] = it.pos0 + div_R(it.rem0 + r0, a.inv_R) + 1;
        tile_hi[qt] = it.pos0 + div_R(it.rem0 + min(r0 + 15, it.rows - 1), a.inv_R) + 1;
      }
      // (rows past the block's last are computed as that row and never written: loads without branches)
      int tok;
      const int idx = row_at(it, min(r0 + (l & 15), it.rows - 1), tok);
      const u32x4* src = reinterpret_cast<const u32x4*>(a.q + (size_t)idx * kD + (l >> 4) * 8);
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) qreg[qt][kk] = src[4 * kk];
    }
  };
  // The queries are waited for here, once: with the loads still pending at the top of the loops the
  // compiler would wait in every step, and for the steps in flight with them.
  auto take_rows = [&] {
#pragma unroll
    for (int qt = 0; qt < kMT; ++qt)
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) {
        qreg[qt][kk] ^= sign_flip;
        asm volatile("" : "+v"(qreg[qt][kk]));
      }
  };
  f32x4 acc[kMT][8];
  float m_run[kMT], l_run[kMT];

  // The stream of steps whose loads are requested, kPfStages - 1 slots ahead of the step that is
  // computed: page ids two at a time by scalar loads, one slot before they are used.  All of it is
  // wave-uniform, and as short as it can be: a scalar instruction costs a wave about as much as a
  // vector instruction (100 of them per step took 170 ns of 870 in a loop of this mix).  A slot past an
  // item's last step repeats that step: its loads fetch valid bytes that nobody uses, so the loop
  // needs no conditional loads and every wait knows how many younger loads are in flight.
  const int32_t* st_table;          // the item's table row
  int st_page, st_first_of_last, st_last, st_left, st_kvh;   // next page, the last step's first page, last page, slots left, KV head
  int r0, r1, r_kvh;                // ids (in flight) and KV head of the slot that is requested next
  uint32_t id_max = 0;              // largest id seen: compared with the pool size once, at the end
  auto start_stream = [&](const PfItem& it) {
    st_table = it.table_row;
    st_page = 2 * it.step0;
    st_last = (it.tok_end - 1) >> 4;
    st_first_of_last = 2 * (it.nsteps - 1);
    st_left = it.slots - it.step0;
    st_kvh = it.kvh;
  };
  auto load_ids = [&] {
    const uint32_t at = (uint32_t)min(st_page, st_first_of_last);
    r0 = ld_uniform_at(st_table, at);
    r1 = ld_uniform_at(st_table, min(at + 1, (uint32_t)st_last));
    r_kvh = st_kvh;
    st_page += 2;
    --st_left;
  };
  // (behind the wait for the step's keys: a wait for LDS data waits for scalar loads in flight as well)
  auto load_ids_after = [&](uint32_t key_word) {
    asm volatile("" : "+s"(st_page) : "v"(key_word));
    load_ids();
  };
  // A step is 1024 16-byte vectors: K of page 0, K of page 1, V of page 0, V of page 1 (256
  // each, contiguous in memory); thread tid fetches vectors tid + k * threads, so which of the
  // four regions a load belongs to is the same for a whole wave: the page's base address is
  // scalar arithmetic and a lane adds only its fixed 32-bit offset.  K lands in LDS as 32 token
  // rows of 256 B with the 16-byte chunk index XOR-ed with a key of the row, V as
  // [page][channel][2 halves of 8 slots] with the unit index XOR-ed with (unit >> 3) & 1, so
  // that the 8 lanes of one operand read hit 8 different bank groups.
  // global_load_lds_dwordx4 moves the vectors from global memory straight into
  // LDS (the 64 lanes of a wave fill 1 KB in lane order, no registers in between).  Wave `wave`
  // fills, for k < kLoads, the 64 slots from slot w0 of region k * kNW/4 + wave/4; the XOR
  // swizzle (an involution inside a key row / a pair of value units) is applied on the source
  // side: the lane that fills slot s fetches vector swz(s).
  static_assert(kNW % 4 == 0, "a wave's 64 vectors must lie in one 256-vector region");
  const int w0 = (wave & 3) * 64;
  uint32_t src_off[kLoads];
  int region[kLoads];
#pragma unroll
  for (int k = 0; k < kLoads; ++k) {
    region[k] = kNW == 4 ? k : k * (kNW / 4) + (wave >> 2);
    const int s_pos = w0 + lane;
    const int slot = s_pos >> 4;
    // swizzle key of K row tau = 16 * (region & 1) + slot: bits 0, 1, 3, 4 of tau (the 16 rows one
    // operand read touches differ in exactly those bits, so its 16 lanes hit 16 different bank groups)
    const int key = ((region[k] & 1) << 3) | ((slot >> 3) << 2) | (slot & 3);
    const int src = (region[k] >> 1) ? (s_pos ^ ((s_pos >> 3) & 1))
                                     : ((slot << 4) | ((s_pos & 15) ^ key));
    src_off[k] = (uint32_t)src * 16;
  }
  auto issue = [&](char* buf) {
    // (an id outside the pool reads page 0)
    id_max = max(id_max, max((uint32_t)r0, (uint32_t)r1));
    const uint32_t p0 = (uint32_t)r0 < (uint32_t)a.num_pages ? r0 : 0, p1 = (uint32_t)r1 < (uint32_t)a.num_pages ? r1 : 0;
    const uint64_t off0 = ((uint64_t)p0 * (uint32_t)a.Hkv + (uint32_t)r_kvh) * (kPage * kD * 2);
    const uint64_t off1 = ((uint64_t)p1 * (uint32_t)a.Hkv + (uint32_t)r_kvh) * (kPage * kD * 2);
#pragma unroll
    for (int k = 0; k < kLoads; ++k) {
      // (scalar base + 32-bit lane offset)
      const GlobalBytes base = reinterpret_cast<GlobalBytes>(reinterpret_cast<uintptr_t>((region[k] >> 1) ? a.v_pages : a.k_pages)) +
                               ((region[k] & 1) ? off1 : off0);
      char* dst = buf + region[k] * 4096 + w0 * 16;   // wave-uniform; lane l lands at dst + 16 l
      __builtin_amdgcn_global_load_lds(
          reinterpret_cast<const __attribute__((address_space(1))) void*>(base + src_off[k]),
          reinterpret_cast<__attribute__((address_space(3))) void*>((uint32_t)reinterpret_cast<uintptr_t>(dst)),
          16, 0, 0);
    }
  };
  const int k_rd = (8 * (i >> 2) + (i & 3)) * 256;
  // value unit 2 * (16 * ct + i) + (j & 1) with its lowest bit XOR-ed: one address for all ct
  const int v_rd = 2 * kBlockTok * kD + (j >> 1) * 4096 + (((2 * i + (j & 1)) ^ ((i >> 2) & 1)) << 4);

  constexpr float kPfRescaleSlack = 8.0f, kPfMaxWeight = 256.0f;   // log2 units; the same as a weight
  constexpr float kLowest = -3.402823466e38f;   // the reference of a row that has seen no key (finite: its weights are exp2(-inf) = 0)
  // One step of 32 keys: all score products, then per tile the exponentials and that tile's output products.
  //   The reference maximum of a row moves only when its weights grow past kPfMaxWeight.  With an
  // exact running maximum one of a wave's 48 rows sets a new record in most steps of a long prompt; with
  // the slack nearly no step after the first moves one, and then neither the rows' maxima nor new
  // references nor rescaled accumulators are needed.  What is tested is the sum of a lane's eight
  // weights, which is formed anyway (no weight exceeds a sum that passes; the eight scores'
  // maximum cost six instructions per tile), and only a step that fails looks for maxima and takes
  // its exponentials again.
  //   kFirst: the item's first step, seen in full by every row.  The rows' maxima come before the only pass, and the
  // accumulators start with this step's products.  The reference has to be the exact maximum here: the weights are rounded to
  // bf16 for the products while their sum is not, and a key that holds much of a row's mass mostly lies in the first step (an
  // attention sink); as the maximum its weight is 1, without rounding.  (With reference 0 where no weight grows too large, half a
  // row's mass on such a key: 1.6e-3 from 64 bits instead of 1.5e-4, 200 to 500 keys.)
  //   kEdge: the causal edge of some row crosses the step, or a tile has no rows; only rows whose maximum exceeds their
  // reference by more than the slack move it.
  enum { kFull, kFirst, kEdge };
  auto compute = [&](const char* buf, auto kind_tag, const int n, const int tok_end, const int (&limit)[kMT]) {
    constexpr int kind = decltype(kind_tag)::value;
    const int t0 = n * kBlockTok;
    u32x4 kr[2][4];
#pragma unroll
    for (int T = 0; T < 2; ++T)
#pragma unroll
      for (int kk = 0; kk < 4; ++kk)
        kr[T][kk] = *reinterpret_cast<const u32x4*>(buf + k_rd + T * 4 * 256 + (((4 * kk + j) ^ i) << 4));
    load_ids_after(kr[1][3][0]);
    f32x4 s0[kMT], s1[kMT];
#pragma unroll
    for (int qt = 0; qt < kMT; ++qt) {
      s0[qt] = f32x4{0.f, 0.f, 0.f, 0.f};
      s1[qt] = f32x4{0.f, 0.f, 0.f, 0.f};
      if (kind == kEdge && t0 >= tile_hi[qt]) continue;   // wave-uniform: no row of the tile sees a token of this step
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) {
        s0[qt] = mfma_16x16x32(kr[0][kk], qreg[qt][kk], s0[qt]);
        s1[qt] = mfma_16x16x32(kr[1][kk], qreg[qt][kk], s1[qt]);
      }
      if (kind == kEdge && t0 + kBlockTok > tile_lo[qt]) {   // wave-uniform: the causal edge crosses this step
        const int sees = limit[qt] - (t0 + 8 * j);           // of this lane's eight keys
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          if (e >= sees) s0[qt][e] = -INFINITY;
          if (4 + e >= sees) s1[qt][e] = -INFINITY;
        }
      }
    }
    u32x4 vr[8];
#pragma unroll
    for (int ct = 0; ct < 8; ++ct) {
      vr[ct] = *reinterpret_cast<const u32x4*>(buf + v_rd + ct * (16 * kPage * 2));
    }
    if (kind == kEdge && t0 + kBlockTok > tok_end) {   // workgroup-uniform; only the last step
      // value slots past the block's last key may hold anything (NaN included): zero them
#pragma unroll
      for (int d = 0; d < 4; ++d) {
        const int tok = t0 + 8 * j + 2 * d;
        const uint32_t mask = (tok < tok_end ? 0x0000ffffu : 0u) | (tok + 1 < tok_end ? 0xffff0000u : 0u);
#pragma unroll
        for (int ct = 0; ct < 8; ++ct) vr[ct][d] &= mask;
      }
    }
#pragma unroll
    for (int qt = 0; qt < kMT; ++qt) {
      if (kind == kEdge && t0 >= tile_hi[qt]) continue;
      float p[8], psum;
      auto row_max = [&] {
        const float mx = fmaxf(fmaxf(fmaxf(s0[qt][0], s0[qt][1]), fmaxf(s0[qt][2], s0[qt][3])),
                               fmaxf(fmaxf(s1[qt][0], s1[qt][1]), fmaxf(s1[qt][2], s1[qt][3])));   // this lane's 8 tokens
        return rows_allreduce_max(mx * sc);
      };
      auto weights = [&] {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          p[e] = __builtin_amdgcn_exp2f(__builtin_fmaf(s0[qt][e], sc, -m_run[qt]));
          p[4 + e] = __builtin_amdgcn_exp2f(__builtin_fmaf(s1[qt][e], sc, -m_run[qt]));
        }
        psum = ((p[0] + p[1]) + (p[2] + p[3])) + ((p[4] + p[5]) + (p[6] + p[7]));
      };
      if (kind == kFirst) m_run[qt] = fmaxf(kLowest, row_max());
      weights();
      if (kind != kFirst && __builtin_amdgcn_ballot_w64(psum > kPfMaxWeight) != 0) {   // wave-uniform
        const float mx = row_max(), m_old = m_run[qt];
        m_run[qt] = kind == kEdge ? (mx > m_old + kPfRescaleSlack ? mx : m_old) : fmaxf(m_old, mx);
        const float alpha = __builtin_amdgcn_exp2f(m_old - m_run[qt]);   // 1 where the row did not move
        l_run[qt] *= alpha;
#pragma unroll
        for (int ct = 0; ct < 8; ++ct) acc[qt][ct] *= alpha;
        weights();
      }
      l_run[qt] = kind == kFirst ? psum : l_run[qt] + psum;
      const u32x4 pb = {pack_bf16(p[0], p[1]), pack_bf16(p[2], p[3]), pack_bf16(p[4], p[5]), pack_bf16(p[6], p[7])};
      const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ct = 0; ct < 8; ++ct) acc[qt][ct] = mfma_16x16x32(vr[ct], pb, kind == kFirst ? zero : acc[qt][ct]);
    }
  };

  // Ring of kPfStages LDS buffers, one slot per step, that runs on from item to item: per slot wait
  // until this wave's part of it has landed (all but the youngest kPfStages-2 slots' loads; stores and
  // query loads in between only make the wait stricter), a bare workgroup barrier (everybody's part has
  // landed and everybody has finished reading the slot before; a fence would wait for every
  // outstanding load), then the loads of the slot kPfStages-1 ahead, which may be the next item's.
  // An item takes at least kPfStages slots, so what is ahead is never further than the next item.
  PfItem cur = first();
  bool more = !kAlone && second < n_ahead;                    // workgroup-uniform: there is a next item
  PfItem nxt = more ? read_item<kSplit>(a, second) : cur;             // (without one its slots are never used)
  int drawn = 0;                                              // (thread 0 only) the item after the next one
  uint32_t ring = 0;                   // byte offset of the current slot's buffer
  constexpr uint32_t kRingBytes = kPfStages * kPfStepBytes;
  static_assert((kRingBytes & (kRingBytes - 1)) == 0, "the ring wraps by a mask");
  start_stream(cur);
#pragma unroll
  for (int s0 = 0; s0 < kPfStages - 1; ++s0) {
    load_ids();
    issue(lds.buf[s0]);
  }
  load_ids();
  load_rows(cur);
  take_rows();
  for (bool drawn_next = false;; drawn_next = true) {
    if (drawn_next) {
      // the next item (the draw was requested before the queries, so it has arrived; as an ordinary store the compiler
      // would put it behind a wait for every load into LDS and every output row that is in flight)
      if (tid == 0) asm volatile("ds_write_b32 %0, %1" :: "v"((uint32_t)reinterpret_cast<uintptr_t>(&lds.next)), "v"(drawn) : "memory");
      __builtin_amdgcn_s_waitcnt(pf_lgkmcnt0);
      asm volatile("" ::: "memory");
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
      const int next = 2 * (int)gridDim.x + __builtin_amdgcn_readfirstlane(lds.next);
      more = next < n_ahead;
      if (more) nxt = read_item<kSplit>(a, next);
    }
    auto ring_step = [&](auto&& comp) {
      __builtin_amdgcn_s_waitcnt(pf_vmcnt_imm((kPfStages - 2) * kLoads));
      asm volatile("" ::: "memory");
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
      issue(lds.buf[0] + ((ring + kRingBytes - kPfStepBytes) & (kRingBytes - 1)));
      if (st_left == 0) start_stream(nxt);                    // (wave-uniform)
      comp(lds.buf[0] + ring);
      ring = (ring + kPfStepBytes) & (kRingBytes - 1);
    };
    // Two loops (their register allocations do not mix): a wave that owns kMT tiles of this block
    // runs the steps before the causal edge of its first tile (tile_lo grows with the tile) in the
    // mask-free code, all other steps in the general code.  Every wave passes the same number of
    // barriers.
    bool all_tiles = true;
#pragma unroll
    for (int qt = 0; qt < kMT; ++qt) all_tiles = all_tiles && (qt * kNW + wave) * 16 < cur.rows;
    const int n_full = all_tiles ? min(tile_lo[0] / kBlockTok, cur.nsteps) : 0;
    int n = cur.step0;
    int limit[kMT] = {};
    if (n < n_full) {
      ring_step([&](const char* buf) { compute(buf, std::integral_constant<int, kFirst>{}, n, 0, limit); });
      for (++n; n < n_full; ++n) ring_step([&](const char* buf) { compute(buf, std::integral_constant<int, kFull>{}, n, 0, limit); });
    } else {
#pragma unroll
      for (int qt = 0; qt < kMT; ++qt) {
        m_run[qt] = kLowest;
        l_run[qt] = 0.f;
#pragma unroll
        for (int ct = 0; ct < 8; ++ct) acc[qt][ct] = f32x4{0.f, 0.f, 0.f, 0.f};
      }
    }
    if (n < cur.nsteps) {
      const int l = opaque_lane();
#pragma unroll
      for (int qt = 0; qt < kMT; ++qt) row_of(cur, qt, l & 15, limit[qt]);
      for (; n < cur.nsteps; ++n) ring_step([&](const char* buf) { compute(buf, std::integral_constant<int, kEdge>{}, n, cur.tok_end, limit); });
    }
    if (more)   // (without a next item nobody waits for the slots that are left)
      for (; n < cur.slots; ++n) ring_step([&](const char*) { load_ids(); });
    // the next item's queries are requested before this item's rows are written
    if (more) {
      // (the pointer is one per lane to the compiler: it would wait at once for the result of an addition that it takes for the wave's)
      int zero = 0;
      asm volatile("" : "+v"(zero));
      if (tid == 0) drawn = atomicAdd(&a.counters[kPfCursor + zero], 1);
      load_rows(nxt);
    }
    const int l2 = opaque_lane();
    // A part of a block's keys: its sums go to memory in the layout of the registers; the workgroup that
    // finds all parts there adds them in their order and writes the rows (nobody waits for another).
    // Stores and loads of the sums carry the device scope (sc1: past the caches that are not shared), and a
    // workgroup counts itself in when its stores are acknowledged.  (With fences, which write back and
    // invalidate caches as a whole, the six chunks took 0.49 ms.)
    bool write_rows = true;
    if (kSplit && cur.split >= 0) {                                    // workgroup-uniform
      const int first = cur.split >> 8, parts = (cur.split & 15) + 1;
      constexpr int kSc1 = 16;
      const auto rs_o = __builtin_amdgcn_make_buffer_rsrc(a.split_o, 0, a.split_bytes, 0x27000);
      // a part's bytes: per wave kMT x 8 fragments of 64 x 16 bytes, then kMT x 64 (maximum, sum)
      constexpr int kWaveBytes = kMT * (8 * 64 * 16 + 64 * 8);
      auto part_at = [&](int k) { return (((first + k) * a.Hkv + cur.kvh) * kNW + wave) * kWaveBytes; };
      {
        const int at = part_at((cur.split >> 4) & 15);
#pragma unroll
        for (int qt = 0; qt < kMT; ++qt) {
#pragma unroll
          for (int ct = 0; ct < 8; ++ct)
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, acc[qt][ct]), rs_o, l2 * 16 + (qt * 8 + ct) * 1024, at, kSc1);
          __builtin_amdgcn_raw_buffer_store_b64(u32x2{__float_as_uint(m_run[qt]), __float_as_uint(l_run[qt])}, rs_o,
                                                l2 * 8 + kMT * 8192 + qt * 512, at, kSc1);
        }
      }
      __builtin_amdgcn_s_waitcnt(pf_vmcnt_imm(0));
      __syncthreads();
      if (tid == 0) lds.arrived = __hip_atomic_fetch_add(a.split_arrived + first * a.Hkv + cur.kvh, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __syncthreads();
      write_rows = __builtin_amdgcn_readfirstlane(lds.arrived) == parts - 1;
      if (write_rows) {
#pragma unroll
        for (int qt = 0; qt < kMT; ++qt) {
          auto ml_of = [&](int k) { return __builtin_amdgcn_raw_buffer_load_b64(rs_o, l2 * 8 + kMT * 8192 + qt * 512, part_at(k), kSc1); };
          float m = -3.402823466e38f;
          for (int k = 0; k < parts; ++k) m = fmaxf(m, __uint_as_float(ml_of(k)[0]));
          l_run[qt] = 0.f;
#pragma unroll
          for (int ct = 0; ct < 8; ++ct) acc[qt][ct] = f32x4{0.f, 0.f, 0.f, 0.f};
          for (int k = 0; k < parts; ++k) {
            const u32x2 ml = ml_of(k);
            u32x4 o[8];
#pragma unroll
            for (int ct = 0; ct < 8; ++ct) o[ct] = __builtin_amdgcn_raw_buffer_load_b128(rs_o, l2 * 16 + (qt * 8 + ct) * 1024, part_at(k), kSc1);
            const float f = __builtin_amdgcn_exp2f(__uint_as_float(ml[0]) - m);
            l_run[qt] = __builtin_fmaf(__uint_as_float(ml[1]), f, l_run[qt]);
#pragma unroll
            for (int ct = 0; ct < 8; ++ct) acc[qt][ct] += __builtin_bit_cast(f32x4, o[ct]) * f;
          }
        }
      }
    }
    // Lane (i, j) holds channels 16*ct + 4*j .. +3 of q-row i.  bf16 rows: the rows of lanes exchange halves of two
    // 16-channel pieces, after which a lane has eight channels in a row and an instruction stores 64 bytes of each of 16 rows.
    // (Through LDS, 128 bytes: the compiler puts a wait for every load into LDS, query and store in flight before a store
    // to LDS, three times 1.4 us per item.)
    auto store_tile = [&](int qt, int out_row) {
      const float inv = 1.0f / rows_allreduce_sum(l_run[qt]);   // a row's sum >= 1: the key that set its reference contributes exp2(0)
      const int j = l2 >> 4;
      if (a.out_dtype == MARL_OUT_F32) {
        float* dst = reinterpret_cast<float*>(a.out) + (size_t)out_row * kD + 4 * j;
        if (out_row >= 0)
#pragma unroll
          for (int ct = 0; ct < 8; ++ct) *reinterpret_cast<f32x4*>(dst + 16 * ct) = acc[qt][ct] * inv;
      } else {
        uint16_t* dst = reinterpret_cast<uint16_t*>(a.out) + (size_t)out_row * kD + 16 * (j & 1) + 8 * (j >> 1);
        u32x4 v[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const f32x4 x = acc[qt][2 * c] * inv, y = acc[qt][2 * c + 1] * inv;
          const auto lo = __builtin_amdgcn_permlane16_swap(pack_bf16(x[0], x[1]), pack_bf16(y[0], y[1]), false, false);
          const auto hi = __builtin_amdgcn_permlane16_swap(pack_bf16(x[2], x[3]), pack_bf16(y[2], y[3]), false, false);
          const uint32_t lo0 = lo[0], lo1 = lo[1], hi0 = hi[0], hi1 = hi[1];
          v[c] = u32x4{lo0, hi0, lo1, hi1};
        }
        if (out_row >= 0)
#pragma unroll
          for (int c = 0; c < 4; ++c) *reinterpret_cast<u32x4*>(dst + 32 * c) = v[c];
      }
    };
    if (write_rows) {
#pragma unroll
      for (int qt = 0; qt < kMT; ++qt) {
        int sees;
        store_tile(qt, row_of(cur, qt, l2 & 15, sees));
      }
    }
    take_rows();
    if (!more) break;
    cur = nxt;
  }
  if (id_max >= (uint32_t)a.num_pages) bad_page = 1;
  __builtin_amdgcn_s_waitcnt(pf_vmcnt_imm(0));   // (the last slots' loads write to LDS: not past the kernel's end)
}

static_assert(sizeof(PrefillLds) <= 80 * 1024, "two workgroups share a CU's 160 KB");
template <bool kSplit>
__global__ __launch_bounds__(kPfThreads)
__attribute__((amdgpu_waves_per_eu(MARL_PREFILL_WAVES_PER_EU, MARL_PREFILL_WAVES_PER_EU)))
void prefill_kernel(PrefillArgs a) {   // kSplit: the list may hold parts of blocks
  __shared__ PrefillLds lds;
  const int grid = (int)gridDim.x;
  const int n_work = *a.list_length * a.Hkv;
  // A workgroup's second item: in a sorted list, and in any of at most two items per workgroup, the longest first items
  // meet the shortest second ones.  (In their order again a prompt of 3008 tokens, 64 / 8 heads, took 161.5 us instead
  // of 150.0, two of up to 3294, 32 / 8 heads, 101.5 instead of 87.7.)  It is not drawn: the counter, asked by all
  // workgroups at their start, delayed their first items (472 items 48.2 -> 43.4 us, 608 items 44.9 -> 40.3 us).
  // A list in group order may end with long blocks: its last two items per workgroup are not bound ahead of time but
  // drawn by whoever has nothing left to do, and start with an empty ring.  (16 prompts of up to 3801 tokens, 16 / 1
  // heads: 377 -> 332 us; 26 of up to 2024, 8 / 2 heads, 156 -> 132; 60 of up to 400, 16 / 1 heads, 63 -> 58.  In
  // sorted lists, whose last items are short, the empty ring costs more than it evens out: 20 prompts of up to 798
  // behind 709, 32 / 8 heads, 143 us, so 165.)
  const bool in_group_order = n_work > 2 * grid && a.counters[kPfIsSorted] == 0;
  const int n_ahead = in_group_order ? max(grid, n_work - 2 * grid) : n_work;
  int first = (int)blockIdx.x, second = in_group_order ? first + grid : 2 * grid - 1 - first;
  int bad_page = 0;
  while (first < n_work) {   // workgroup-uniform
    // (the arguments are read again for each run: kept through the loop they would cost the registers of another
    // twenty spilled values)
    auto kernarg = __builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(kernarg));
    const PrefillArgs run = *(const PrefillArgs*)kernarg;
    if (kSplit && run.counters[kPfDivided] != 0) prefill_items<true, false>(run, [&] { return read_item<true>(run, first); }, second, n_ahead, lds, bad_page);
    else prefill_items<false, false>(run, [&] { return read_item<false>(run, first); }, second, n_ahead, lds, bad_page);
    if (!in_group_order) break;
    if (threadIdx.x == 0) lds.late = n_ahead + atomicAdd(&a.counters[kPfLate], 1);
    __syncthreads();   // (the loads of slots past the end have landed: prefill_items ends with their wait)
    first = __builtin_amdgcn_readfirstlane(lds.late);
    second = n_work;
  }
  if (bad_page) atomicOr(&a.counters[kPfFlags], MARL_FLAG_BAD_PAGE);
}

// Small calls in one launch: no order, no parts, an item per workgroup, which finds its block in the groups by itself.  What bounds
// it is the chain of dependent loads at its start (groups, page ids, keys): 4 us of the 7 of the smallest call; the plan, a launch
// of its own before the items, took as long again.
// The first workgroup sets the flags, by the groups and the page ids that they address: nobody
// else writes that word, which no earlier kernel has cleared.
__global__ __launch_bounds__(kPfThreads)
__attribute__((amdgpu_waves_per_eu(MARL_PREFILL_WAVES_PER_EU, MARL_PREFILL_WAVES_PER_EU)))
void prefill_small_kernel(PrefillArgs a) {
  __shared__ PrefillLds lds;
  __shared__ FindLds find;
  if (blockIdx.x == 0) {
    int flag = 0;
    if (threadIdx.x == 0) find.flags = 0;
    walk_groups(a, 0x7fffffff, flag, find, [&](int g, int n, int, int) {   // (all groups: those past the room for blocks are flagged, too)
      const int32_t* row = a.prefix_table + (size_t)g * a.max_pp;
      const int last = (a.q_pos0[g] + n - 1) / kPage;
      constexpr int kIds = 8;          // of a group, requested together
      for (int p = 0; p <= last; p += kIds) {
        int id[kIds];
#pragma unroll
        for (int u = 0; u < kIds; ++u) id[u] = row[min(p + u, last)];
#pragma unroll
        for (int u = 0; u < kIds; ++u) flag |= (unsigned)id[u] >= (unsigned)a.num_pages ? MARL_FLAG_BAD_PAGE : 0;
      }
    });
    __syncthreads();
    if (flag) atomicOr(&find.flags, flag);
    __syncthreads();
    if (threadIdx.x == 0) a.counters[kPfFlags] = find.flags;
    return;
  }
  const int item = (int)blockIdx.x - 1, block = item / a.Hkv;
  int g, packed, bad_page = 0;
  if (find_block(a, block, g, packed, find))   // workgroup-uniform
    prefill_items<false, true>(a, [&] { return item_of<false>(a, block, item - block * a.Hkv, g, packed); }, 0, 0, lds, bad_page);
}

// Scatter of a prompt chunk's keys and values into the group's pages: column `col` of group g's table row, whose chunk brings n
// tokens from q row b on to position pos0, for one KV head and 128 threads.  The key rows of a page are contiguous
// (4 KB): 16-byte copies.  Values are stored channel-major, so thread c collects channel c of the page's 16 tokens and writes
// its 32 bytes with two stores when the chunk covers the whole page, else slot by slot.
// What bounds it: memory (256 prompts, 1.36 GB read and written: 274 us, 5 TB/s), a short call its launch and three dependent reads.
__device__ __forceinline__ void write_prompt_page(const PrefillArgs& a, const int g, const int b, const int n, const int pos0,
                                                  const int kvh, const int col) {
  const int c = threadIdx.x;
  const int lo = max(pos0, col * kPage), hi = min(pos0 + n, (col + 1) * kPage);   // positions to write
  const int page = a.prefix_table[(size_t)g * a.max_pp + col];
  if ((unsigned)page >= (unsigned)a.num_pages) {
    if (kvh == 0 && c == 0 && a.flags) atomicOr(a.flags, MARL_FLAG_BAD_PAGE);
    return;
  }
  const size_t blk = ((size_t)page * a.Hkv + kvh) * (kPage * kD);                 // elements
  const size_t tok0 = (size_t)b + (col * kPage - pos0);                           // token of slot 0 (may be "negative")
  const size_t row_stride = (size_t)a.Hkv * kD;
  // keys: 16 slots x 16 chunks of 16 bytes, two per thread
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const int v = c + k * kD;
    const int slot = v >> 4, chunk = v & 15;
    const int pos = col * kPage + slot;
    if (pos >= lo && pos < hi)
      *reinterpret_cast<u32x4*>(a.k_pages_w + blk + (size_t)slot * kD + chunk * 8) =
          *reinterpret_cast<const u32x4*>(a.k_new + (tok0 + slot) * row_stride + (size_t)kvh * kD + chunk * 8);
  }
  // values: channel c of every slot
  uint16_t vals[kPage];
#pragma unroll
  for (int slot = 0; slot < kPage; ++slot) {
    const int pos = col * kPage + slot;
    vals[slot] = (pos >= lo && pos < hi) ? a.v_new[(tok0 + slot) * row_stride + (size_t)kvh * kD + c] : (uint16_t)0;
  }
  uint16_t* vdst = a.v_pages_w + blk + (size_t)c * kPage;
  if (hi - lo == kPage) {
    u32x4 w0, w1;
#pragma unroll
    for (int d = 0; d < 4; ++d) {
      w0[d] = (uint32_t)vals[2 * d] | ((uint32_t)vals[2 * d + 1] << 16);
      w1[d] = (uint32_t)vals[8 + 2 * d] | ((uint32_t)vals[8 + 2 * d + 1] << 16);
    }
    *reinterpret_cast<u32x4*>(vdst) = w0;
    *reinterpret_cast<u32x4*>(vdst + 8) = w1;
  } else {
#pragma unroll
    for (int slot = 0; slot < kPage; ++slot) {
      const int pos = col * kPage + slot;
      if (pos >= lo && pos < hi) vdst[slot] = vals[slot];
    }
  }
}

// `cols` workgroups per (group, KV head): one for every column of the tables, or else for every so many-th of those that the chunk
// touches, from the first on.
template <bool kAll>
__global__ __launch_bounds__(kD) void kv_write_prompt_kernel(PrefillArgs a, int cols) {
  const int at = blockIdx.x % cols;
  const int gk = blockIdx.x / cols;
  const int g = gk / a.Hkv, kvh = gk % a.Hkv;
  int flag = 0;
  const int n = group_tokens(a, g, flag);
  const int pos0 = a.q_pos0[g];
  if (at == 0 && kvh == 0 && threadIdx.x == 0 && flag && a.flags) atomicOr(a.flags, flag);
  if (n == 0) return;
  const int first = (int)((unsigned)pos0 / kPage), last = (int)((unsigned)(pos0 + n - 1) / kPage);
  if (kAll) {
    if (at >= first && at <= last) write_prompt_page(a, g, a.q_start[g], n, pos0, kvh, at);
  } else {
#pragma unroll 1
    for (int col = first + at; col <= last; col += cols) write_prompt_page(a, g, a.q_start[g], n, pos0, kvh, col);
  }
}

// Where the chunks touch few of the columns: a workgroup for every page that they may touch together, and KV head.  A group whose
// tokens begin at row b has the places from b / 16 + 2 g on: n tokens touch at most n / 16 + 2 pages, so that groups that share
// no rows share no place, and the last place lies before NT / 16 + 2 NG, which the host knows.  Which group a place belongs to
// the workgroup finds by itself: it looks at all of them (0.2 us of the call for 70, 0.7 for 210, 1.9 for 500), and so writes every group's pages
// whatever the order of q_start.
constexpr int kScatterGroups = 1024;
__global__ __launch_bounds__(kD) void kv_write_prompt_pages_kernel(PrefillArgs a) {
  extern __shared__ int4 chunk_of[];                     // [NG] first row, tokens, position, first column less its place
  __shared__ unsigned long long here[kScatterGroups / 64];
  const int place = blockIdx.x / a.Hkv, kvh = blockIdx.x % a.Hkv;
  const int c = threadIdx.x, lane = c & 63;
  int flag = 0;
  // the group's first row, tokens, position and first column less its place; whether this workgroup's place is one of its pages
  auto chunk = [&](int g, int4& h) {
    h = make_int4(0, 0, 0, 0);
    if (g >= a.NG) return false;
    const int n = group_tokens(a, g, flag), b = a.q_start[g], pos0 = a.q_pos0[g];
    const int first = (int)((unsigned)pos0 / kPage), shift = first - (int)((unsigned)b / kPage + 2u * (unsigned)g);
    h = make_int4(b, n, pos0, shift);
    return n > 0 && place + shift >= first && place + shift <= (int)((unsigned)(pos0 + n - 1) / kPage);
  };
  if (a.NG <= 64) {                                      // a wave sees them all: no LDS, no barrier
    int4 h;
    const bool mine = chunk(lane, h);
    if (blockIdx.x == 0 && c < 64 && flag && a.flags) atomicOr(a.flags, flag);
    for (unsigned long long m = __builtin_amdgcn_ballot_w64(mine); m != 0; m &= m - 1) {   // (one group, unless groups share rows)
      const int g = __builtin_ctzll(m);
      write_prompt_page(a, g, __builtin_amdgcn_readlane(h.x, g), __builtin_amdgcn_readlane(h.y, g),
                        __builtin_amdgcn_readlane(h.z, g), kvh, place + __builtin_amdgcn_readlane(h.w, g));
    }
    return;
  }
  for (int g0 = 0; g0 < a.NG; g0 += kD) {                // workgroup-uniform
    const int g = g0 + c;
    int4 h;
    const unsigned long long m = __builtin_amdgcn_ballot_w64(chunk(g, h));
    if (g < a.NG) chunk_of[g] = h;
    if (lane == 0) here[g >> 6] = m;
  }
  if (blockIdx.x == 0 && flag && a.flags) atomicOr(a.flags, flag);
  __syncthreads();
  for (int w = 0; w < (a.NG + 63) / 64; ++w) {           // workgroup-uniform
    unsigned long long m = here[w];
    m = (unsigned long long)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(m >> 32)) << 32 |
        (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)m);
    for (; m != 0; m &= m - 1) {
      const int g = 64 * w + __builtin_ctzll(m);
      const int4 h = chunk_of[g];
      write_prompt_page(a, g, __builtin_amdgcn_readfirstlane(h.x), __builtin_amdgcn_readfirstlane(h.y),
                        __builtin_amdgcn_readfirstlane(h.z), kvh, place + __builtin_amdgcn_readfirstlane(h.w));
    }
  }
}

}  // namespace

int prefill_rows_per_block() { return kQB; }

PrefillSplitLayout prefill_split_layout(long max_blocks, long Hkv, long max_keys) {
  PrefillSplitLayout L = {};
  if (max_blocks > kPfSorted || max_keys <= kPfLongKeys) return L;   // (the plan divides nothing then)
  L.entries = kPfSorted;
  L.parts = (int)std::min<long>(kPfMaxParts, max_blocks * kPfMaxDiv * std::min<long>(Hkv, kPfMaxParts));
  L.bytes = (size_t)L.parts * kNW * kMT * 64 * (sizeof(float2) + 8 * sizeof(f32x4));   // (about 100 MB at most)
  return L;
}

int prefill_blocks_per_cu() {
  int n = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, prefill_kernel<true>, kPfThreads, 0) != hipSuccess || n < 1) n = 1;
  return n;
}

// Whether a call is taken by one launch without a plan.  Not where the plan would weigh parts; what can be known here are the bounds
// of the number of items and of their keys.  Up to as many items as run at the same time it is always faster (planned / here, us: one
// prompt of 45 tokens, 28 / 4 heads, 11.4 and 7.0; 12 of up to 362, 31.1 and 25.7; 19 of up to 151, 32 / 8, 21.0 and 14.8).  Beyond that the
// order of the items, and each one's start while another runs, are worth more as items get longer and more of them share a
// workgroup: with at most 448 keys and six items per workgroup none of 60 random calls was slower (19.1 and 11.3; 42.8 and
// 35.6 for 1400 items of up to 67 keys; 93 and 88 for 3700 of up to 200), behind it some (10 prompts of up to 731, 28 / 4 heads, 39.6 and
// 42.3; 40 of up to 503, 8 / 2, 30.8 and 32.7; 5000 items of up to 162 keys 109 and 116, 11000 of up to 70 183 and 215).
// The keys are those that a table row can hold: rows of a fixed capacity above 960 tokens keep their calls on the plan, however short
// the prompts are.
constexpr long kPfSmallRounds = 6, kPfSmallKeys = 448;
static bool is_small_prefill(const PrefillArgs& a) {
  const long items = (long)a.max_blocks * a.Hkv, keys = (long)a.max_pp * kPage;
  return keys <= kPfLongKeys && (items < a.slots || (items <= kPfSmallRounds * a.slots && keys <= kPfSmallKeys));
}

hipError_t launch_prefill(const PrefillArgs& a, int grid, hipStream_t st) {
  if (is_small_prefill(a)) {
    hipLaunchKernelGGL(prefill_small_kernel, dim3((unsigned)(a.max_blocks * a.Hkv + 1)), dim3(kPfThreads), 0, st, a);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(prefill_plan_kernel, dim3(1), dim3(kPlanThreadsPf), 0, st, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (a.split_slots > 0) hipLaunchKernelGGL(prefill_kernel<true>, dim3(grid), dim3(kPfThreads), 0, st, a);
  else hipLaunchKernelGGL(prefill_kernel<false>, dim3(grid), dim3(kPfThreads), 0, st, a);
  return hipGetLastError();
}

hipError_t launch_kv_write_prompt(const PrefillArgs& a, hipStream_t st) {
  if (a.NT == 0 || a.NG == 0) return hipSuccess;
  // How long a chunk is the host does not know, only what there is together and how wide the tables are.
  //   1. Every column that a chunk may touch has a workgroup where that leaves few without work (0.3 us a thousand), or where
  // memory hides them: 256 chunks of up to 1500, 64 / 8 heads, 364 us, by places 400; 900 of up to 600 behind up to 300 556 and 931.
  //   2. Twice the mean of the chunks' columns, and a longer chunk's workgroups go round (1.1 us each time), where the longest that there
  // can be takes less than an eighth of what the call needs for its bytes: 400 of up to 1000 behind up to 3000, 64 / 8, 402 us by
  // columns, 397 by rounds, 426 by places.
  //   3. Else the places: one chunk of 8192 tokens and 31 of one, 16 / 1 heads, 8.9 us by columns, 23 by rounds, 4.2 by places,
  // 64 / 8 54, 38 and 12; one of 300 and 40 of one, 28 / 4, 4.9, 10.2 and 4.9; 200 single tokens behind up to 4000, 64 / 8, 126, 10 and 6.8; six of up to 512 behind up to 8192,
  // 64 / 8, 14.7, 8.2 and 7.3.  (Groups without end would cost each workgroup more than the rounds do.)
  const long all = std::min<long>(a.max_pp, a.NT / kPage + 2);       // columns that a chunk may touch
  const long places = a.NT / kPage + 2l * a.NG;
  const long mean = (a.NT + (long)a.NG * kPage - 1) / ((long)a.NG * kPage);
  const bool few_empty = a.NG * all * a.Hkv <= 2048 || a.NG * all <= (places * a.Hkv >= 8192 ? 4 : 2) * places;
  long cols = few_empty ? all : std::min(all, 2 * mean + 2);
  const bool short_rounds = (all + cols - 1) / cols * (8 * 1100) <= places * a.Hkv * 3;   // ns; 16 KB at 5 TB/s a place and head
  if (few_empty || short_rounds || a.NG > kScatterGroups)
    hipLaunchKernelGGL(cols == a.max_pp ? kv_write_prompt_kernel<true> : kv_write_prompt_kernel<false>, dim3((unsigned)(a.NG * a.Hkv * cols)), dim3(kD), 0, st, a, (int)cols);
  else
    hipLaunchKernelGGL(kv_write_prompt_pages_kernel, dim3((unsigned)(places * a.Hkv)), dim3(kD), a.NG <= 64 ? 0 : sizeof(int4) * a.NG, st, a);
  return hipGetLastError();
}

}  // namespace marl
