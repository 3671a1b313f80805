// Decode attention of a small call (the general kernels are in attn_kernels.hip): a workgroup takes all tokens,
// prefix and own, of one (sequence, KV head), its waves take the 32-token steps in turn, and the combined rows are
// final, so one launch does it.  Of long rows several workgroups take a part of the steps each, and a second
// launch adds the parts.  The call's plan (which the header promises in the workspace) is built by one more workgroup
// of the first launch; nobody waits for it.
//
// What bounds it: latency (launch, group id -> prefix length -> page id -> keys, the combine), and from about 512
// tokens per workgroup on what one CU can have in flight (70 GB/s; eight waves instead of four take the same
// time).  The general kernels' three or four dependent launches (plan 5, prefix 9, merge 9 us of kernel time at the first
// size) pass the work list and the partials through memory.  A prefix is read once per sequence here and not once per
// group; the L2s serve that (see the order of the workgroups below).  Measured per call, general kernels and this one:
// 16 sequences in 4 groups, 8 / 2 heads, 256 + 128 tokens: 22.0 and 8.1 us (6.4 since the plan looks at padded page tables in
// pieces and the binding's calls are lighter); 32 heads' worth of items with 4096 + 4096 tokens: 45 and 19 us (8
// parts); 256 sequences in 64 groups, 8 / 2 heads, 1024 + 1024 tokens: 66 and 42 us.
//
// Wave-level scheme as in attn_kernels.hip (v_mfma_f32_16x16x32_bf16, K and V straight into operand registers).
#include <algorithm>
#include <type_traits>

#include "marl_internal.h"
#include "plan_lds.h"
#include "wave_ops.h"

namespace marl {
namespace {

constexpr int NW = kAttnThreads / 64;
constexpr int kAccRowFloats = kD + 4;   // (the 16 rows that a wave instruction writes start in different banks)
constexpr int kSeqBlock = 8;            // sequences whose workgroups for one KV head and part run on one XCD

struct SmallLds {
  float m[NW][16];
  float l[NW][16];
  __attribute__((aligned(16))) float acc[NW][16][kAccRowFloats];
};

typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ void store_row_piece(const AttnArgs& a, size_t at, f32x4 v) {
  if (a.out_dtype == MARL_OUT_F32) {
    *reinterpret_cast<f32x4*>(reinterpret_cast<float*>(a.out) + at) = v;
  } else {
    *reinterpret_cast<bf16x4*>(reinterpret_cast<uint16_t*>(a.out) + at) = bf16x4{(__bf16)v[0], (__bf16)v[1], (__bf16)v[2], (__bf16)v[3]};
  }
}

// Tokens of part `part` of (sequence s, KV head kvh): final rows, or with several parts partials in slots 0 .. splits - 1.
__device__ __forceinline__ void small_item(const AttnArgs& a, const int s, const int kvh, const int part) {
  __shared__ SmallLds lds;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int i = lane & 15, j = lane >> 4;
  const float sc = fmaxf(fabsf(a.scale) * 1.44269504088896340736f, 1e-30f);
  const uint32_t sign_flip = a.scale < 0.f ? 0x80008000u : 0u;

  const int g = ld_uniform(a.group_of_seq + s);
  const int S = min(max(ld_uniform(a.suffix_lens + s), 0), a.max_sp * kPage);
  // Q^T operand: lane (i, j) holds channels 8*(4*kk + j) .. +8 of query row i
  u32x4 qreg[4];
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) {
    u32x4 v = {0u, 0u, 0u, 0u};
    if (i < a.R) v = *reinterpret_cast<const u32x4*>(a.q + ((size_t)s * a.Hq + kvh * a.R + i) * kD + (4 * kk + j) * 8);
    qreg[kk] = v ^ sign_flip;
  }
  const bool grouped = (unsigned)g < (unsigned)a.NG;
  const int P = grouped ? min(max(ld_uniform(a.prefix_lens + g), 0), a.max_pp * kPage) : 0;
  const int32_t* prefix_row = a.prefix_table + (size_t)(grouped ? g : 0) * a.max_pp;
  const int32_t* suffix_row = a.suffix_table + (size_t)s * a.max_sp;
  // steps: those of the prefix, then those of the sequence's own tokens
  const int prefix_steps = (P + kBlockTok - 1) / kBlockTok;
  const int all_steps = prefix_steps + (S + kBlockTok - 1) / kBlockTok;
  const int first_step = (int)((long)all_steps * part / a.splits), steps = (int)((long)all_steps * (part + 1) / a.splits);

  f32x4 acc[8];
  float m_run = -INFINITY, l_run = 0.f;
#pragma unroll
  for (int ct = 0; ct < 8; ++ct) acc[ct] = f32x4{0.f, 0.f, 0.f, 0.f};

  const size_t page_bytes = (size_t)a.Hkv * (kPage * kD * 2);
  const char* kbase = reinterpret_cast<const char*>(a.k_pages) + (size_t)kvh * (kPage * kD * 2) +
                      ((8 * ((i >> 2) & 1) + (i & 3)) * (kD * 2) + j * 16);
  const char* vbase = reinterpret_cast<const char*>(a.v_pages) + (size_t)kvh * (kPage * kD * 2) +
                      (i * (kPage * 2) + (j & 1) * 16);
  // Page ids (scalar loads) of step k and how many of its tokens exist.  An id outside the pool reads page 0 (the
  // plan's workgroup raises the flag).
  auto load_pages = [&](int k, int& p0, int& p1, int& tokens) {
    const bool own = k >= prefix_steps;
    const int t = (own ? k - prefix_steps : k) * kBlockTok;
    const int32_t* row = (own ? suffix_row : prefix_row) + (t >> 4);
    tokens = (own ? S : P) - t;
    p0 = ld_uniform(row);
    p1 = tokens > kPage ? ld_uniform(row + 1) : p0;
    if ((unsigned)p0 >= (unsigned)a.num_pages) p0 = 0;
    if ((unsigned)p1 >= (unsigned)a.num_pages) p1 = 0;
  };
  u32x4 kr[2][4], vr[8];
  auto issue_k = [&](int p0, int p1) {
    const char* kp = kbase + (size_t)(i < 8 ? p0 : p1) * page_bytes;
#pragma unroll
    for (int T = 0; T < 2; ++T)
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) kr[T][kk] = *reinterpret_cast<const u32x4*>(kp + T * (4 * kD * 2) + kk * 64);
  };
  auto issue_v = [&](int p0, int p1) {
    const char* vp = vbase + (size_t)(j < 2 ? p0 : p1) * page_bytes;
#pragma unroll
    for (int ct = 0; ct < 8; ++ct) vr[ct] = *reinterpret_cast<const u32x4*>(vp + ct * (16 * kPage * 2));
  };

  // K registers are refilled for the wave's next step as soon as the score products have consumed them, V
  // registers after the output products; the last step is peeled, so that the loop has no conditional loads.
  int k = first_step + wave, tokens = 0, n0 = 0, n1 = 0, ntokens = 0;
  auto step = [&](auto has_next_tag) {
    constexpr bool kHasNext = decltype(has_next_tag)::value;
    f32x4 sv[2];
#pragma unroll
    for (int T = 0; T < 2; ++T) {
      sv[T] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) sv[T] = mfma_16x16x32(kr[T][kk], qreg[kk], sv[T]);
    }
    if constexpr (kHasNext) issue_k(n0, n1);
    if (tokens < kBlockTok) {   // wave-uniform: the end of the prefix or of the own tokens
      // tokens past the end: score -inf (weight 0), and zero their value slots, which may hold anything
#pragma unroll
      for (int T = 0; T < 2; ++T)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (8 * j + 4 * T + e >= tokens) sv[T][e] = -INFINITY;
#pragma unroll
      for (int d = 0; d < 4; ++d) {
        const int tok = 8 * j + 2 * d;
        const uint32_t mask = (tok < tokens ? 0x0000ffffu : 0u) | (tok + 1 < tokens ? 0xffff0000u : 0u);
#pragma unroll
        for (int ct = 0; ct < 8; ++ct) vr[ct][d] &= mask;
      }
    }
    float mx = fmaxf(fmaxf(fmaxf(sv[0][0], sv[0][1]), fmaxf(sv[0][2], sv[0][3])),
                     fmaxf(fmaxf(sv[1][0], sv[1][1]), fmaxf(sv[1][2], sv[1][3])));
    mx = rows_allreduce_max(mx);
    const float m_new = fmaxf(m_run, mx * sc);
    const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);
    float p[8];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      p[e] = __builtin_amdgcn_exp2f(__builtin_fmaf(sv[0][e], sc, -m_new));
      p[4 + e] = __builtin_amdgcn_exp2f(__builtin_fmaf(sv[1][e], sc, -m_new));
    }
    const float psum = ((p[0] + p[1]) + (p[2] + p[3])) + ((p[4] + p[5]) + (p[6] + p[7]));
    if (__builtin_amdgcn_ballot_w64(m_new > m_run) != 0) {   // wave-uniform
#pragma unroll
      for (int ct = 0; ct < 8; ++ct) acc[ct] *= alpha;
    }
    l_run = l_run * alpha + psum;
    m_run = m_new;
    const u32x4 pb = {pack_bf16(p[0], p[1]), pack_bf16(p[2], p[3]), pack_bf16(p[4], p[5]), pack_bf16(p[6], p[7])};
#pragma unroll
    for (int ct = 0; ct < 8; ++ct) acc[ct] = mfma_16x16x32(vr[ct], pb, acc[ct]);
    if constexpr (kHasNext) {
      issue_v(n0, n1);
      tokens = ntokens;
      k += NW;
      if (k + NW < steps) load_pages(k + NW, n0, n1, ntokens);
    }
  };
  if (k < steps) {   // wave-uniform
    load_pages(k, n0, n1, tokens);
    issue_k(n0, n1);
    issue_v(n0, n1);
    if (k + NW < steps) load_pages(k + NW, n0, n1, ntokens);
    while (k + NW < steps) step(std::true_type{});
    step(std::false_type{});
  }

  // the waves' results, combined in wave order (bit-identical reruns)
  l_run = rows_allreduce_sum(l_run);
  if (j == 0) {
    lds.m[wave][i] = m_run;
    lds.l[wave][i] = l_run;
  }
#pragma unroll
  for (int ct = 0; ct < 8; ++ct) *reinterpret_cast<f32x4*>(&lds.acc[wave][i][16 * ct + 4 * j]) = acc[ct];
  __syncthreads();
  for (int e = threadIdx.x; e < a.R * (kD / 4); e += NW * 64) {
    const int r = e / (kD / 4), c4 = e % (kD / 4);
    float mm = lds.m[0][r];
#pragma unroll
    for (int w = 1; w < NW; ++w) mm = fmaxf(mm, lds.m[w][r]);
    float ll = 0.f;
    f32x4 o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const float mw = lds.m[w][r];
      const float f = (mw == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(mw - mm);
      ll = __builtin_fmaf(lds.l[w][r], f, ll);
      o += *reinterpret_cast<const f32x4*>(&lds.acc[w][r][4 * c4]) * f;
    }
    if (a.splits > 1) {
      const size_t slot = ((size_t)s * a.Hq + kvh * a.R + r) * (a.NCp + a.NCs) + part;
      *reinterpret_cast<f32x4*>(a.partial_o + slot * kD + 4 * c4) = o;
      if (c4 == 0) a.partial_ml[slot] = make_float2(mm, ll);
      continue;
    }
    f32x4 res = {0.f, 0.f, 0.f, 0.f};
    if (ll > 0.f) res = o * (1.0f / ll);   // (no token at all: zeros)
    store_row_piece(a, ((size_t)s * a.Hq + kvh * a.R + r) * kD + 4 * c4, res);
  }
}

// Workgroups are dealt to the eight XCDs in turn.  The workgroups of eight neighbouring sequences (usually samples of
// one prompt) for one KV head and part follow each other on one XCD, so that the prefix they share is read out
// of its L2: 64 groups of 4 samples, 16 / 2 heads, 2304 tokens: 67 -> 41 us against a plain order.  The last block of sequences
// comes after the others and is as wide as there are sequences left: with empty workgroups for those that are not there, the
// others met on a few CUs of the XCD (one sequence, 8 KV heads, 131072 tokens: 282 us, now 112; 4 KV heads, 16384: 25.7, now 16.9).
struct SmallGrid {
  int units;        // (KV head, part) pairs of a block of sequences
  int left;         // sequences of the last, narrower block
  int full_slots;   // of an XCD: workgroups for blocks of kSeqBlock sequences (the last eight units may be past the end)
  __host__ __device__ SmallGrid(const AttnArgs& a)
      : units(a.Hkv * a.splits), left(a.NS % kSeqBlock), full_slots((a.NS / kSeqBlock * units + 7) / 8 * kSeqBlock) {}
  __host__ __device__ int workgroups() const { return 8 * (full_slots + (units + 7) / 8 * left); }
};

__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 3)))
void decode_small_kernel(AttnArgs a) {
  if (blockIdx.x == 0) {
    plan_in_lds<kAttnThreads, kSmallAttnSeqs, kSmallAttnSeqs, int, true>(a);
    return;
  }
  const SmallGrid g(a);
  const int xcd = (blockIdx.x - 1) & 7, slot = (blockIdx.x - 1) >> 3;
  int unit = slot / kSeqBlock * 8 + xcd, first = 0, at = slot % kSeqBlock, end = a.NS - g.left;
  if (slot >= g.full_slots) {   // workgroup-uniform
    unit = (slot - g.full_slots) / g.left * 8 + xcd;
    at = (slot - g.full_slots) % g.left;
    first = end;
    end = a.NS;
  }
  const int part = unit % a.splits, pair = unit / a.splits;
  const int s = first + pair / a.Hkv * kSeqBlock + at;
  if (s < end) small_item(a, s, pair % a.Hkv, part);   // (the last units may be past the end)
}

// Parts of a row added in their order (half a wave per row): the formula of the general merge kernel.
__global__ __launch_bounds__(kAttnThreads) void merge_parts_kernel(AttnArgs a) {
  const int row = blockIdx.x * (kAttnThreads / 32) + (threadIdx.x >> 5);
  if (row >= a.NS * a.Hq) return;
  const int sub = threadIdx.x & 31;   // channels 4 sub .. + 3
  const size_t slot = (size_t)row * (a.NCp + a.NCs);
  const float2* ml = a.partial_ml + slot;
  const float* po = a.partial_o + slot * kD + 4 * sub;
  constexpr int kAtOnce = 4;   // parts requested together
  float mstar = -INFINITY, denom = 0.f;
  f32x4 sum = {0.f, 0.f, 0.f, 0.f};
  for (int k0 = 0; k0 < a.splits; k0 += kAtOnce) {
    float2 v[kAtOnce];
    f32x4 o[kAtOnce];
#pragma unroll
    for (int u = 0; u < kAtOnce; ++u) {
      const int k = min(k0 + u, a.splits - 1);
      v[u] = ml[k];
      o[u] = *reinterpret_cast<const f32x4*>(po + (size_t)k * kD);
      if (k0 + u >= a.splits) v[u].x = -INFINITY;
    }
    float mn = mstar;
#pragma unroll
    for (int u = 0; u < kAtOnce; ++u) mn = fmaxf(mn, v[u].x);
    const float f0 = mstar == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mstar - mn);
    denom *= f0;
    sum *= f0;
#pragma unroll
    for (int u = 0; u < kAtOnce; ++u) {
      const float f = v[u].x == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(v[u].x - mn);
      denom = __builtin_fmaf(v[u].y, f, denom);
      sum += o[u] * f;
    }
    mstar = mn;
  }
  f32x4 res = {0.f, 0.f, 0.f, 0.f};
  if (denom > 0.f) res = sum * (1.0f / denom);
  store_row_piece(a, (size_t)row * kD + 4 * sub, res);
}

}  // namespace

// Which calls these are: judged by what the table rows can hold (lengths stay on the device).  The lines are drawn
// where the general kernels begin to win, which read a prefix once per group and balance long rows: 3978 random
// batches of 1 to 512 sequences, 1 to 32 samples per prompt, all head counts of the tests and up to 4 M tokens x KV heads
// were timed with both.  Up to 1.5 M of them, of which 1 M may be prefix, 6 of 2788 batches lose more than 3 % and the mean
// gain is 2.1 times; at 2 M and 1.3 M 16 of 3055 lose, the worst 0.72 times.
// Parts: none below 1024 tokens (the second launch costs 3 us: 8 against 11 us), else of 384 tokens, as long as
// at most 1536 workgroups come of it (768 run at a time; 768 or 512 in all lose 2-4 %, as lengths differ), and at most 16 of a
// row: what the second launch adds up grows with them, and is paid by what a table can hold (8 sequences of 40 tokens in rows for
// 131072, one KV head: 8.9 us, 10.5 with 32 parts, 14.3 with 64; 10 pairs of 16384: 19.1, 23.5, 23.1), while one
// to four pairs of long rows would gain (one of 16384: 15.5, 12.9, 13.5; of 131072: 79, 45, 33).
int small_attn_splits(const AttnArgs& a) {
  const long items = (long)a.NS * a.Hkv, prefix = (long)a.max_pp * kPage, own = (long)a.max_sp * kPage;
  if (a.NS > kSmallAttnSeqs || a.NG > kSmallAttnSeqs || items > 1l << 16) return 0;
  if (items * (prefix + own) > 3l << 19 || items * prefix > 1l << 20) return 0;
  if (prefix + own < 1024) return 1;
  const long n = std::min({(prefix + own) / 384, 1536 / items, 16l, (long)a.NCp + a.NCs});
  return (int)std::max(n, 1l);
}

hipError_t launch_small_attn(const AttnArgs& a, hipStream_t st) {
  const int grid = SmallGrid(a).workgroups() + 1;   // (at most 65536 pairs and 1536 parts: see above)
  hipLaunchKernelGGL(decode_small_kernel, dim3(grid), dim3(kAttnThreads), 0, st, a);
  return hipGetLastError();
}

hipError_t launch_merge_parts(const AttnArgs& a, hipStream_t st) {
  constexpr int kRows = kAttnThreads / 32;
  hipLaunchKernelGGL(merge_parts_kernel, dim3((a.NS * a.Hq + kRows - 1) / kRows), dim3(kAttnThreads), 0, st, a);
  return hipGetLastError();
}

}  // namespace marl
