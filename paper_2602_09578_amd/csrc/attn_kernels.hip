// Decode attention over the paged KV cache: the prefix kernel (a group's prefix KV is
// streamed once and applied to all of the group's query rows), the suffix kernel (each
// sequence's own generated tokens) and the merge kernel.  The first two produce
// flash-decoding style partials (running max, running sum, unnormalised output) per (query
// row, chunk of tokens), which the merge kernel combines; a sequence whose own tokens are a
// single work item is finished by whoever processes that item instead.  Calls of medium size have prefix and
// suffix items in one kernel (the items kernel), where a long item behind a prefix is a partial too.  (Small calls:
// attn_small_kernel.hip.)
//
// Context in the paper: rollout is memory-bound on KV caches (Section 4.1), every prompt is
// expanded into several samples that share its prefix (Section 5.1) and lengths are skewed
// (Section 2.2); the paper gives no kernel, so the design below is this library's own.
//
// Wave-level scheme (gfx950, wave64, v_mfma_f32_16x16x32_bf16).  A wave handles 32 tokens
// (two pages) per step and up to MT tiles of 16 query rows.  Lane l = 16*j + i.
//   scores:  D[token-row][q-row] = K-tile (A operand) x Q^T (B operand).  A-row i of tile T
//            is the token 8*(i/4) + 4*T + i%4 of the 32, so that after both tiles lane
//            (i, j) holds the scores of q-row i for tokens 8j..8j+7: exactly the B operand
//            layout the second product needs, with no data movement.
//   output:  D[channel][q-row] += V^T-tile (A operand) x P^T (B operand), 8 channel tiles.
//            V pages are stored [channel][slot], so lane (i, j) loads its 8 tokens of
//            channel 16*ct + i with one 16-byte load.
// Suffix kernel: K and V go straight from global memory into MFMA operand registers (16-byte
// loads; per instruction a wave reads 16 x 64 B of K or 2 x 512 B of V); LDS only combines
// the four waves of a workgroup, which split the item's tokens between them.
// Prefix kernel: the four waves split the query rows instead and share each K/V step
// through a ring of LDS tiles (described at the kernel).
#include <algorithm>
#include <type_traits>

#include "marl_internal.h"
#include "wave_ops.h"

namespace marl {
namespace {

constexpr int kWaves = kAttnThreads / 64;
constexpr int kMaximaAtOnce = 8;   // of partials that are about to be added

// LDS per workgroup for the cross-wave combine: (max, sum) and the row index of every q-row, and
// every wave's accumulators in row-major order (a row is 128 floats, padded to 132 so that the
// 16 rows a wave instruction writes start in different banks).
constexpr int kAccRowFloats = kD + 4;
template <int MT>
struct ItemLds {
  float m[kWaves][MT * 16];
  float l[kWaves][MT * 16];
  int row[MT * 16];
  __attribute__((aligned(16))) float acc[kWaves][MT * 16][kAccRowFloats];
};

// Processes tokens [tok_begin, tok_end) of one block-table row for MT tiles of query rows
// and writes one partial per valid row.  NW is the number of waves that share the item:
//   NW = 4: called by all four waves of the workgroup, which take the 32-token steps in
//           turn and are combined through LDS (workgroup barriers inside);
//   NW = 1: called by one wave on its own (no LDS, no barrier): for short items.
//   row_index[qt]: for this lane's q-row (i) of tile qt, seq*Hq + head, or -1 if the row
//   does not exist.  slot: partial slot of this chunk.
//   finish (uniform over the callers): the item holds all of the sequence's own tokens, so the
//   rows' only other partials are the n_prefix_partials prefix partials of its group, which an
//   earlier kernel has completed: they are merged with the item's own result (the merge
//   kernel's formula and order: prefix slots first) and the final output rows are written
//   instead of a partial.
template <int MT, int NW>
__device__ __forceinline__ void process_item(const AttnArgs& a, const int32_t* __restrict__ table_row,
                                             const int tok_begin, const int tok_end, const int kvh,
                                             const int (&row_index)[MT], const int slot,
                                             ItemLds<MT>& lds, int& bad_page,
                                             const bool finish = false, const int n_prefix_partials = 0) {
  const int lane = threadIdx.x & 63;
  const int wave = NW == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int i = lane & 15, j = lane >> 4;
  // scores are kept in log2 units; a zero scale becomes a tiny one so that -inf * sc stays -inf
  const float sc = fmaxf(fabsf(a.scale) * 1.44269504088896340736f, 1e-30f);
  const uint32_t sign_flip = a.scale < 0.f ? 0x80008000u : 0u;
  const int nslot = a.NCp + a.NCs;

  // Q^T operand: lane (i, j) holds channels 8*(4*kk + j) .. +8 of q-row i
  u32x4 qreg[MT][4];
  auto ready_q = [&] {
#pragma unroll
    for (int qt = 0; qt < MT; ++qt)
#pragma unroll
      for (int kk = 0; kk < 4; ++kk)
#pragma unroll
        for (int e = 0; e < 4; ++e) qreg[qt][kk][e] = row_index[qt] >= 0 ? qreg[qt][kk][e] ^ sign_flip : 0u;
  };
#pragma unroll
  for (int qt = 0; qt < MT; ++qt) {
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      if constexpr (NW == 1) {   // without a branch, and used only once the first keys and values are requested too
        qreg[qt][kk] = *reinterpret_cast<const u32x4*>(a.q + (size_t)max(row_index[qt], 0) * kD + (4 * kk + j) * 8);
      } else {
        u32x4 v = {0u, 0u, 0u, 0u};
        if (row_index[qt] >= 0) {
          v = *reinterpret_cast<const u32x4*>(a.q + (size_t)row_index[qt] * kD + (4 * kk + j) * 8);
          v ^= sign_flip;
        }
        qreg[qt][kk] = v;
      }
    }
  }

  f32x4 acc[MT][8];
  float m_run[MT], l_run[MT];
#pragma unroll
  for (int qt = 0; qt < MT; ++qt) {
    m_run[qt] = -INFINITY;
    l_run[qt] = 0.f;
#pragma unroll
    for (int ct = 0; ct < 8; ++ct) acc[qt][ct] = f32x4{0.f, 0.f, 0.f, 0.f};
  }

  const size_t page_bytes = (size_t)a.Hkv * (kPage * kD * 2);
  const char* kbase = reinterpret_cast<const char*>(a.k_pages) + (size_t)kvh * (kPage * kD * 2) +
                      ((8 * ((i >> 2) & 1) + (i & 3)) * (kD * 2) + j * 16);
  const char* vbase = reinterpret_cast<const char*>(a.v_pages) + (size_t)kvh * (kPage * kD * 2) +
                      (i * (kPage * 2) + (j & 1) * 16);

  // Page ids of the 32-token step that starts at token t (wave-uniform, scalar loads).
  auto load_pages = [&](int t, int& p0, int& p1) {
    p0 = ld_uniform(table_row + (t >> 4));
    p1 = (t + kPage < tok_end) ? ld_uniform(table_row + (t >> 4) + 1) : p0;
    if ((unsigned)p0 >= (unsigned)a.num_pages) { p0 = 0; bad_page = 1; }
    if ((unsigned)p1 >= (unsigned)a.num_pages) { p1 = 0; bad_page = 1; }
  };
  u32x4 kr[2][4], vr[8];
  auto issue_k = [&](int p0, int p1) {
    const char* kp = kbase + (size_t)(i < 8 ? p0 : p1) * page_bytes;
#pragma unroll
    for (int T = 0; T < 2; ++T)
#pragma unroll
      for (int kk = 0; kk < 4; ++kk)
        kr[T][kk] = ld_stream_k(kp + T * (4 * kD * 2) + kk * 64);
  };
  auto issue_v = [&](int p0, int p1) {
    const char* vp = vbase + (size_t)(j < 2 ? p0 : p1) * page_bytes;
#pragma unroll
    for (int ct = 0; ct < 8; ++ct) vr[ct] = ld_stream(vp + ct * (16 * kPage * 2));
  };

  // Software pipeline: the K registers are refilled for the next step as soon as the score
  // MFMAs have consumed them, the V registers as soon as the output MFMAs have; page ids are
  // fetched one step ahead.  So a wave keeps 16 KB of loads in flight while it computes.
  // The last step of a wave is peeled (no refill; it alone can be ragged) so that the loop
  // body has no conditional loads and every wait leaves the younger 8 loads in flight.
  constexpr int stride = NW * kBlockTok;
  int t0 = tok_begin + wave * kBlockTok;
  int tn = t0 + stride;
  int n0 = 0, n1 = 0;

  // a one-wave item's first prefix partial: max and sum with the queries, values in the place of the last keys
  float2 ml0 = make_float2(-INFINITY, 0.f);
  f32x4 o0[8];
  const float* const o0_src = a.partial_o + (size_t)max(row_index[0], 0) * nslot * kD + 4 * j;
  if constexpr (NW == 1) {
    if (finish && n_prefix_partials > 0) ml0 = a.partial_ml[(size_t)max(row_index[0], 0) * nslot];
  }

  auto step = [&](auto has_next_tag) {
    constexpr bool kHasNext = decltype(has_next_tag)::value;
    f32x4 s[MT][2];
#pragma unroll
    for (int qt = 0; qt < MT; ++qt)
#pragma unroll
      for (int T = 0; T < 2; ++T) {
        s[qt][T] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) s[qt][T] = mfma_16x16x32(kr[T][kk], qreg[qt][kk], s[qt][T]);
      }
    if constexpr (kHasNext) issue_k(n0, n1);

    if constexpr (!kHasNext) {
      if constexpr (NW == 1) {
        if (finish && n_prefix_partials > 0) {   // wave-uniform
#pragma unroll
          for (int ct = 0; ct < 8; ++ct) o0[ct] = *reinterpret_cast<const f32x4*>(o0_src + 16 * ct);
        }
      }
      if (t0 + kBlockTok > tok_end) {   // wave-uniform: the ragged end of a chunk
        // tokens past the end: score -inf (weight 0), and zero their value slots, which may
        // hold anything (NaN included)
#pragma unroll
        for (int qt = 0; qt < MT; ++qt)
#pragma unroll
          for (int T = 0; T < 2; ++T)
#pragma unroll
            for (int e = 0; e < 4; ++e)
              if (t0 + 8 * j + 4 * T + e >= tok_end) s[qt][T][e] = -INFINITY;
#pragma unroll
        for (int d = 0; d < 4; ++d) {
          const int tok = t0 + 8 * j + 2 * d;
          const uint32_t mask = (tok < tok_end ? 0x0000ffffu : 0u) | (tok + 1 < tok_end ? 0xffff0000u : 0u);
#pragma unroll
          for (int ct = 0; ct < 8; ++ct) vr[ct][d] &= mask;
        }
      }
    }

    u32x4 pb[MT];
#pragma unroll
    for (int qt = 0; qt < MT; ++qt) {
      const f32x4 s0 = s[qt][0], s1 = s[qt][1];
      float mx = fmaxf(fmaxf(fmaxf(s0[0], s0[1]), fmaxf(s0[2], s0[3])),
                       fmaxf(fmaxf(s1[0], s1[1]), fmaxf(s1[2], s1[3])));
      mx = rows_allreduce_max(mx);
      const float m_new = fmaxf(m_run[qt], mx * sc);
      const float alpha = __builtin_amdgcn_exp2f(m_run[qt] - m_new);
      float p[8];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        p[e] = __builtin_amdgcn_exp2f(__builtin_fmaf(s0[e], sc, -m_new));
        p[4 + e] = __builtin_amdgcn_exp2f(__builtin_fmaf(s1[e], sc, -m_new));
      }
      const float psum = ((p[0] + p[1]) + (p[2] + p[3])) + ((p[4] + p[5]) + (p[6] + p[7]));
      if (__builtin_amdgcn_ballot_w64(m_new > m_run[qt]) != 0) {   // wave-uniform
#pragma unroll
        for (int ct = 0; ct < 8; ++ct) acc[qt][ct] *= alpha;
      }
      l_run[qt] = l_run[qt] * alpha + psum;
      m_run[qt] = m_new;
      pb[qt] = u32x4{pack_bf16(p[0], p[1]), pack_bf16(p[2], p[3]), pack_bf16(p[4], p[5]), pack_bf16(p[6], p[7])};
    }
#pragma unroll
    for (int ct = 0; ct < 8; ++ct)
#pragma unroll
      for (int qt = 0; qt < MT; ++qt) acc[qt][ct] = mfma_16x16x32(vr[ct], pb[qt], acc[qt][ct]);

    if constexpr (kHasNext) {
      issue_v(n0, n1);
      t0 = tn;
      tn += stride;
      if (tn < tok_end) load_pages(tn, n0, n1);
    }
  };

  if (t0 < tok_end) {
    load_pages(t0, n0, n1);
    issue_k(n0, n1);
    issue_v(n0, n1);
    if (tn < tok_end) load_pages(tn, n0, n1);
    if constexpr (NW == 1) ready_q();
    while (tn < tok_end) step(std::true_type{});
    step(std::false_type{});
  }

  // the four lanes that share a q-row each hold a part of its sum
#pragma unroll
  for (int qt = 0; qt < MT; ++qt) {
    l_run[qt] = rows_allreduce_sum(l_run[qt]);
  }

  if constexpr (NW > 1) {
    // Combine the waves: every wave puts its (max, sum) and its accumulators, row-major, into
    // LDS; after one barrier all threads share the 16 x 128 outputs, each computing a float4 as
    // the sum over the waves in wave order (fixed order: bit-identical reruns) rescaled to the
    // common max, and the workgroup writes every row's 512 bytes as full cache lines.
    static_assert(MT == 1, "the workgroup-wide combine handles one 16-row tile");
    if (j == 0) {
      lds.m[wave][i] = m_run[0];
      lds.l[wave][i] = l_run[0];
      if (wave == 0) lds.row[i] = row_index[0];
    }
#pragma unroll
    for (int ct = 0; ct < 8; ++ct)
      *reinterpret_cast<f32x4*>(&lds.acc[wave][i][16 * ct + 4 * j]) = acc[0][ct];
    __syncthreads();
    constexpr int kPerThread = 16 * (kD / 4) / (NW * 64);   // float4 outputs per thread
#pragma unroll
    for (int k = 0; k < kPerThread; ++k) {
      const int e = threadIdx.x + k * NW * 64;
      const int r = e / (kD / 4), c4 = e % (kD / 4);
      const int ridx = lds.row[r];
      if (ridx >= 0) {
        float mm = lds.m[0][r];
#pragma unroll
        for (int w = 1; w < NW; ++w) mm = fmaxf(mm, lds.m[w][r]);
        float ll = 0.f;
        f32x4 o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < NW; ++w) {
          const float mw = lds.m[w][r];
          const float f = (mw == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(mw - mm);
          ll += lds.l[w][r] * f;
          o += *reinterpret_cast<const f32x4*>(&lds.acc[w][r][4 * c4]) * f;
        }
        if (!finish) {
          const size_t ps = (size_t)ridx * nslot + slot;
          *reinterpret_cast<f32x4*>(a.partial_o + ps * kD + 4 * c4) = o;
          if (c4 == 0) a.partial_ml[ps] = make_float2(mm, ll);
        } else {
          const size_t p0 = (size_t)ridx * nslot;
          float mstar = mm;
          for (int k = 0; k < n_prefix_partials; ++k) mstar = fmaxf(mstar, a.partial_ml[p0 + k].x);
          float denom = 0.f;
          f32x4 sum = {0.f, 0.f, 0.f, 0.f};
          for (int k = 0; k < n_prefix_partials; ++k) {
            const float2 v = a.partial_ml[p0 + k];
            const f32x4 ok = *reinterpret_cast<const f32x4*>(a.partial_o + (p0 + k) * kD + 4 * c4);
            const float f = (v.x == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(v.x - mstar);
            denom = __builtin_fmaf(v.y, f, denom);
            sum += ok * f;
          }
          {
            const float f = (mm == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(mm - mstar);
            denom = __builtin_fmaf(ll, f, denom);
            sum += o * f;
          }
          f32x4 res = {0.f, 0.f, 0.f, 0.f};
          if (denom > 0.f) res = sum * (1.0f / denom);
          if (a.out_dtype == MARL_OUT_F32) {
            *reinterpret_cast<f32x4*>(reinterpret_cast<float*>(a.out) + (size_t)ridx * kD + 4 * c4) = res;
          } else {
            typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
            const bf16x4 v = {(__bf16)res[0], (__bf16)res[1], (__bf16)res[2], (__bf16)res[3]};
            *reinterpret_cast<bf16x4*>(reinterpret_cast<uint16_t*>(a.out) + (size_t)ridx * kD + 4 * c4) = v;
          }
        }
      }
    }
    // the next use of this LDS comes after the workgroup's next trip to the work queue, which
    // has barriers of its own
  } else {
    // one wave on its own: lane (i, j) holds channels 16*ct + 4*j .. +3 of q-row i
#pragma unroll
    for (int qt = 0; qt < MT; ++qt) {
      if (row_index[qt] >= 0) {
        if (!finish) {
          const size_t ps = (size_t)row_index[qt] * nslot + slot;
          float* dst = a.partial_o + ps * kD + 4 * j;
#pragma unroll
          for (int ct = 0; ct < 8; ++ct) *reinterpret_cast<f32x4*>(dst + 16 * ct) = acc[qt][ct];
          if (j == 0) a.partial_ml[ps] = make_float2(m_run[qt], l_run[qt]);
        } else {
          const size_t p0 = (size_t)row_index[qt] * nslot;
          float mstar = fmaxf(m_run[qt], ml0.x);
          for (int k = 1; k < n_prefix_partials; k += kMaximaAtOnce) {
            float mk[kMaximaAtOnce];
#pragma unroll
            for (int u = 0; u < kMaximaAtOnce; ++u) mk[u] = a.partial_ml[p0 + min(k + u, n_prefix_partials - 1)].x;
#pragma unroll
            for (int u = 0; u < kMaximaAtOnce; ++u) mstar = fmaxf(mstar, mk[u]);
          }
          float denom = 0.f;
          f32x4 sum[8];
#pragma unroll
          for (int ct = 0; ct < 8; ++ct) sum[ct] = f32x4{0.f, 0.f, 0.f, 0.f};
          if (n_prefix_partials > 0) {
            const float f = (ml0.x == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(ml0.x - mstar);
            denom = __builtin_fmaf(ml0.y, f, denom);
#pragma unroll
            for (int ct = 0; ct < 8; ++ct) sum[ct] += o0[ct] * f;
          }
          for (int k = 1; k < n_prefix_partials; ++k) {
            const float2 v = a.partial_ml[p0 + k];
            const float f = (v.x == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(v.x - mstar);
            denom = __builtin_fmaf(v.y, f, denom);
            const float* src = a.partial_o + (p0 + k) * kD + 4 * j;
#pragma unroll
            for (int ct = 0; ct < 8; ++ct) sum[ct] += *reinterpret_cast<const f32x4*>(src + 16 * ct) * f;
          }
          {
            const float f = (m_run[qt] == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(m_run[qt] - mstar);
            denom = __builtin_fmaf(l_run[qt], f, denom);
#pragma unroll
            for (int ct = 0; ct < 8; ++ct) sum[ct] += acc[qt][ct] * f;
          }
          const float inv = denom > 0.f ? 1.0f / denom : 0.f;
#pragma unroll
          for (int ct = 0; ct < 8; ++ct) {
            const f32x4 res = sum[ct] * inv;
            const size_t at = (size_t)row_index[qt] * kD + 16 * ct + 4 * j;
            if (a.out_dtype == MARL_OUT_F32) {
              *reinterpret_cast<f32x4*>(reinterpret_cast<float*>(a.out) + at) = res;
            } else {
              typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
              const bf16x4 v = {(__bf16)res[0], (__bf16)res[1], (__bf16)res[2], (__bf16)res[3]};
              *reinterpret_cast<bf16x4*>(reinterpret_cast<uint16_t*>(a.out) + at) = v;
            }
          }
        }
      }
    }
  }
}

// ---------------------------------------------------------------------------------------
// Suffix kernels: one work item = (sequence, chunk of its generated tokens, KV head); the
// R = Hq/Hkv query heads of that KV head are the (zero-padded) 16-row tile.
//
// The item list is sorted longest first, so it splits into a head of long items (more than
// kShortTokens tokens) and a tail of short ones.
//   suffix_kernel:       long items, one per workgroup (waves take the 32-token steps in
//                        turn), taken from the queue only when the workgroup is free
//                        (reserving an item early would undo the longest-first balancing).
//   short_suffix_items:  short items, one per wave, split round-robin over all waves of the
//                        grid with no LDS traffic, barrier or atomic, so a batch of tiny
//                        sequences does not pay a workgroup's fixed costs per sequence.
//                        Where they run: a sequence whose own tokens are one short item (the
//                        usual case) is finished in the first phase of the MERGE kernel, after
//                        the prefix partials are complete: its rows never pass through a partial.
//                        The short items of sequences with several suffix chunks must be
//                        partials before the merge kernel starts: they run as the first phase of
//                        the PREFIX (or items) kernel's workgroups (as a phase of the suffix kernel they
//                        slowed the long items' hot loop down by a few percent through the
//                        shared register allocation, and a kernel of their own cost one more
//                        launch per call).
// ---------------------------------------------------------------------------------------
#ifndef MARL_SUFFIX_WAVES_PER_EU
#define MARL_SUFFIX_WAVES_PER_EU 3
#endif
#ifndef MARL_SUFFIX_WAVES
#define MARL_SUFFIX_WAVES 4
#endif
constexpr int kSuffixWaves = MARL_SUFFIX_WAVES;   // waves that share one long item (= workgroup size / 64)
__global__ __launch_bounds__(kSuffixWaves * 64)
__attribute__((amdgpu_waves_per_eu(MARL_SUFFIX_WAVES_PER_EU, MARL_SUFFIX_WAVES_PER_EU)))
void suffix_kernel(AttnArgs a) {
  __shared__ ItemLds<1> lds;
  __shared__ int next_item;
  const int n_work = a.counters[MARL_CTR_NUM_LONG_SUFFIX_ITEMS] * a.Hkv;
  int bad_page = 0;
  // the first item of a workgroup is its block index (no trip to the shared counter, on which
  // a whole grid starting at once would queue up); later ones come from the counter
  for (bool first = true;; first = false) {
    int qi = blockIdx.x;
    if (!first) {
      if (n_work <= (int)gridDim.x) break;   // every item has a workgroup of its own: no draw
      if (threadIdx.x == 0) next_item = gridDim.x + atomicAdd(&a.counters[MARL_CTR_SUFFIX_CURSOR], 1);
      __syncthreads();
      qi = next_item;
      __syncthreads();
    }
    if (qi >= n_work) break;
    const int4 it = a.suffix_items[qi / a.Hkv];
    const int kvh = qi % a.Hkv;
    const int s = it.x;
    const int i = threadIdx.x & 15;
    const int row_index[1] = {i < a.R ? s * a.Hq + kvh * a.R + i : -1};
    // a sequence whose own tokens are this one item: the output rows are finished here
    const int chunks = ld_uniform(a.seq_chunks + s);
    process_item<1, kSuffixWaves>(a, a.suffix_table + (size_t)s * a.max_sp, it.y, it.z, kvh, row_index,
                                  a.NCp + it.y / a.Cs, lds, bad_page, (chunks >> 16) == 1, chunks & 0xffff);
  }
  if (bad_page) atomicOr(&a.counters[MARL_CTR_FLAGS], MARL_FLAG_BAD_PAGE);
}

// Short suffix items: wave w of the grid takes the entries n_long + w, n_long + w + W, ...
// (W = waves in the grid) with no LDS, no barrier and no atomic: the entries are sorted by
// size, so a round-robin split is balanced, and a shared queue counter would serialise
// thousands of waves on one address.  The next record is fetched while the current item runs.
// kFinish = false (first phase of the prefix and items kernels): the items of sequences with several
// suffix chunks, as partials.  kFinish = true (first phase of the merge kernel, after the
// prefix partials are complete): the items of sequences whose own tokens are that one item,
// finished to output rows, so that they never travel through a partial.
// What bounds a finished item is its chain of dependent loads (record, page ids, keys and values of each step, prefix partials)
// with three waves per SIMD; what these keep in flight is 5 TB/s (32768 items) to 6.5 (8192), of the 7.0 of plain reading.  So nothing waits between the queries' request and the keys', and the first prefix partial is under way
// while the last step is computed, in the last keys' registers (with the queries it had spilled): 8192 sequences of 40 tokens
// behind 256, 28 / 4 heads, 228 -> 220 us (1.0 GB); of up to 60 behind 64: 200 -> 193; 64 x 32 of up to 64 behind 4096: 50.4 ->
// 47.  (Records and page ids an item ahead, in three workgroups per CU that stay: the same to 1 us.)
template <bool kFinish>
__device__ __forceinline__ void short_suffix_items(const AttnArgs& a, int& bad_page) {
  const int n_long = a.counters[MARL_CTR_NUM_LONG_SUFFIX_ITEMS] * a.Hkv;
  const int n_work = a.counters[MARL_CTR_NUM_SUFFIX_ITEMS] * a.Hkv;
  const int waves_per_block = blockDim.x >> 6;
  const int stride = gridDim.x * waves_per_block;
  int cur = n_long + blockIdx.x * waves_per_block + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (cur >= n_work) return;
  const int i = threadIdx.x & 15;
  int4 rec = a.suffix_items[cur / a.Hkv];
  while (cur < n_work) {
    const int nxt = cur + stride;
    const int4 nrec = nxt < n_work ? a.suffix_items[nxt / a.Hkv] : make_int4(0, 0, 0, 0);
    const int kvh = cur % a.Hkv;
    const int s = rec.x;
    const int chunks = ld_uniform(a.seq_chunks + s);
    if (((chunks >> 16) == 1) == kFinish) {
      const int row_index[1] = {i < a.R ? s * a.Hq + kvh * a.R + i : -1};
      ItemLds<1>* no_lds = nullptr;   // the one-wave path never touches it
      process_item<1, 1>(a, a.suffix_table + (size_t)s * a.max_sp, rec.y, rec.z, kvh, row_index,
                         a.NCp + rec.y / a.Cs, *no_lds, bad_page, kFinish, chunks & 0xffff);
    }
    cur = nxt;
    rec = nrec;
  }
}

// ---------------------------------------------------------------------------------------
// Prefix kernel: one work item = (group, chunk of prefix tokens, block of up to 128 (or 256)
// query rows, KV head); two kernels, one for each block size.  Query row rho of a group is (its
// rho / R -th sequence, head kvh*R + rho % R).
//
// Here the four waves split the QUERY rows (16-row tile t belongs to wave t % 4) and every wave sees
// all tokens, so the group's K/V must reach all of them: each 32-token step (two pages, 16 KB of K and V)
// is fetched once by the workgroup with fully coalesced 16-byte loads (a wave reads 1 KB contiguous
// per instruction) into a ring of LDS tiles and read back in MFMA operand layout.  No cross-wave
// reduction is needed.
//
// LDS tile of one step (16 KB): K as 32 token rows of 256 B, the 16-byte chunk index of
// row tau XOR-ed with a 4-bit key made of bits 0, 1, 3, 4 of tau: the 16 rows that the 16 lanes
// of one operand read touch differ in exactly those bits, so they hit 16 different 16-byte bank
// groups (measured: 4.1 cycles per wave instruction per CU against 7.3 with a 3-bit key, 4.0 for
// a plain linear read); V as [page][channel][2 halves of 8 slots], the 16-byte unit index u
// XOR-ed with (u>>3)&1 for the same reason.
// ---------------------------------------------------------------------------------------
constexpr int kStepBytes = 2 * kBlockTok * kD * 2;   // K + V of one 32-token step
// prefix items rescale their accumulators only when a lane's eight weights sum to more than this
constexpr float kMaxWeight = 256.0f;
// s_waitcnt immediate (gfx9 encoding): vector-memory counter <= vm, LDS/scalar counter <= lgkm
constexpr int waitcnt_imm(int vm, int lgkm) { return (vm & 0xf) | ((vm >> 4) << 14) | (7 << 4) | ((lgkm & 0xf) << 8); }
// Data path of an item: global memory straight into an LDS ring of four steps
// (global_load_lds_dwordx4, the swizzle of the LDS tile applied on the source side, no staging registers)
// -> operand registers.  Iteration n: wait for slot n+1, workgroup barrier; loads of slot n+3; read V(n);
// score products of step n (K(n) is in registers); read K(n+1) into the K registers; softmax of step n,
// which covers both reads; output products.  No LDS read is waited for where it is issued.
//   Blocks of 256 rows, bound by instructions: a row's reference maximum moves only when a lane's eight
// weights sum to more than kMaxWeight (no weight exceeds a sum that passes), a branch taken in the first
// step and hardly ever after.  Blocks of 128 rows, bound by memory, keep the exact running maximum: a row's
// largest weight is then 1, which bf16 holds exactly.
//   Blocks of up to 256 rows (kHalves) are taken by two workgroups, half of the row tiles each, that run
// on the same XCD, usually on the same CU: the second reads the group's keys and values out of the L2
// (so these are ordinary cached loads), and each SIMD has two waves that no barrier keeps in step (one
// waits or runs its softmax while the other feeds the matrix core).  Blocks of up to 128 rows stream
// their keys and values once, with non-temporal loads (cached: 131 -> 141 and 343 -> 386 us on the first two
// lists below).
//   What bounds it, blocks of 128 rows: HBM, and on short lists the latency of an item's start and of its
// steps.  256 groups of 8 samples x 7 rows, 512-2048 shared tokens: 131 us (5.4 TB/s); 64 groups of 4 x 8
// rows, 8192 tokens: 343 us (6.5 TB/s), as with staging through registers; 4 groups of 16 x 8 rows, 512-2048
// tokens: 28.8 -> 26.7 us, 4 groups of 4 x 4 rows, 256 tokens: 12.2 -> 10.1 us.  Blocks of 256 rows: issue of
// matrix and vector instructions (180 flop per byte): 64 groups of 32 samples x 7 rows on 4096 shared tokens
// 177 -> 150 us (0.80 PFLOP/s); the 177 us were one workgroup of 8 waves per CU with all of a group's rows,
// staged through registers and kept in step by one barrier per step.
constexpr int kPrefixStages = 4;
struct PrefixLds {
  __attribute__((aligned(16))) char buf[kPrefixStages][kStepBytes];
};
typedef const char __attribute__((address_space(1))) * GlobalBytes;

template <bool kHalves>
__device__ __forceinline__ void prefix_item(const AttnArgs& a, const int4 it, const int kvh, const int half,
                                            PrefixLds& lds, int& bad_page) {
  constexpr int NW = 4, MTW = 2, kLoads = 4;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int i = lane & 15, j = lane >> 4;
  const int g = it.x, tok_begin = it.y, tok_end = it.z;
  // this half's tiles: a block of at most eight tiles is not divided (its keys are then read once)
  constexpr int kBlockRows = kHalves ? kRowsPerQBlockWide : kRowsPerQBlock;
  const int nrows = ld_uniform(a.group_count + g) * a.R;
  const int gstart = ld_uniform(a.group_start + g);
  const int tiles_all = (min(kBlockRows, nrows - it.w) + 15) >> 4;
  const int tiles0 = tiles_all <= MTW * NW ? tiles_all : (tiles_all + 1) >> 1;
  const int tiles = half ? tiles_all - tiles0 : tiles0;
  if (kHalves && tiles <= 0) return;                         // workgroup-uniform (a first half is never empty)
  const int row_begin = it.w + (half ? tiles0 * 16 : 0);
  const int nt = tiles > wave + NW ? 2 : tiles > wave ? 1 : 0;   // wave-uniform: tiles wave, wave + 4

  const int32_t* table_row = a.prefix_table + (size_t)g * a.max_pp;
  const int nsteps = (tok_end - tok_begin + kBlockTok - 1) / kBlockTok;
  const int first_page = tok_begin >> 4;
  const int last_page = (tok_end - 1) >> 4;
  // Page ids (scalar): fetched an iteration before they are used, checked once per item.  A slot past
  // the end repeats the last page: valid bytes that nobody uses, so that every wait knows how many
  // loads are in flight.
  uint32_t id_max = 0;
  int r0, r1;
  auto fetch_ids = [&](int n) {
    r0 = ld_uniform(table_row + min(first_page + 2 * n, last_page));
    r1 = ld_uniform(table_row + min(first_page + 2 * n + 1, last_page));
  };
  // A step is 1024 16-byte vectors: K of page 0, K of page 1, V of page 0, V of page 1 (256 each,
  // contiguous in memory); wave w fills slots 64 w .. + 63 of each region, in lane order.  K as 32 token
  // rows of 256 B, the 16-byte chunk index XOR-ed with bits 0, 1, 3, 4 of the row; V as [page][channel][2
  // halves of 8 slots], the unit index u XOR-ed with (u >> 3) & 1: both are undone on the source side.
  uint32_t src_off[kLoads];
#pragma unroll
  for (int k = 0; k < kLoads; ++k) {
    const int s_pos = wave * 64 + lane;
    const int slot = s_pos >> 4;
    const int key = ((k & 1) << 3) | ((slot >> 3) << 2) | (slot & 3);
    src_off[k] = 16u * (uint32_t)((k >> 1) ? (s_pos ^ ((s_pos >> 3) & 1)) : ((slot << 4) | ((s_pos & 15) ^ key)));
  }
  auto issue = [&](uint32_t ring) {
    id_max = max(id_max, max((uint32_t)r0, (uint32_t)r1));
    const uint32_t p0 = (uint32_t)r0 < (uint32_t)a.num_pages ? r0 : 0, p1 = (uint32_t)r1 < (uint32_t)a.num_pages ? r1 : 0;
    const uint64_t off0 = ((uint64_t)p0 * (uint32_t)a.Hkv + (uint32_t)kvh) * (kPage * kD * 2);
    const uint64_t off1 = ((uint64_t)p1 * (uint32_t)a.Hkv + (uint32_t)kvh) * (kPage * kD * 2);
#pragma unroll
    for (int k = 0; k < kLoads; ++k) {
      const GlobalBytes base = reinterpret_cast<GlobalBytes>(reinterpret_cast<uintptr_t>((k >> 1) ? a.v_pages : a.k_pages)) +
                               ((k & 1) ? off1 : off0);
      char* dst = lds.buf[0] + (ring + k * 4096 + wave * 1024);   // wave-uniform; lane l lands at dst + 16 l
      __builtin_amdgcn_global_load_lds(
          reinterpret_cast<const __attribute__((address_space(1))) void*>(base + src_off[k]),
          reinterpret_cast<__attribute__((address_space(3))) void*>((uint32_t)reinterpret_cast<uintptr_t>(dst)), 16, 0, kHalves ? 0 : 2);   // (2: non-temporal)
    }
  };
  constexpr uint32_t kRingBytes = kPrefixStages * kStepBytes;
  static_assert((kRingBytes & (kRingBytes - 1)) == 0, "the ring wraps by a mask");
  // the first three steps are requested before the chain of dependent loads that leads to the query rows
#pragma unroll
  for (int s0 = 0; s0 < kPrefixStages - 1; ++s0) {
    fetch_ids(s0);
    issue(s0 * kStepBytes);
  }
  fetch_ids(kPrefixStages - 1);

  const float sc = fmaxf(fabsf(a.scale) * 1.44269504088896340736f, 1e-30f);
  const uint32_t sign_flip = a.scale < 0.f ? 0x80008000u : 0u;
  const int nslot = a.NCp + a.NCs;
  const int slot = tok_begin / a.Cp;
  int row_index[MTW];
  u32x4 qreg[MTW][4];
#pragma unroll
  for (int qt = 0; qt < MTW; ++qt) {
    const int rho = row_begin + (qt * NW + wave) * 16 + i;
    int idx = -1;
    if (qt < nt && rho < nrows) idx = a.group_seqs[gstart + rho / a.R] * a.Hq + kvh * a.R + rho % a.R;
    row_index[qt] = idx;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      u32x4 v = {0u, 0u, 0u, 0u};
      if (idx >= 0) v = *reinterpret_cast<const u32x4*>(a.q + (size_t)idx * kD + (4 * kk + j) * 8);
      v ^= sign_flip;
      qreg[qt][kk] = v;
    }
  }
  // (waited for here, once: with loads pending at the top of the loop the compiler would wait in every
  // step, and for the steps in flight with them)
#pragma unroll
  for (int qt = 0; qt < MTW; ++qt)
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) asm volatile("" : "+v"(qreg[qt][kk]));
  f32x4 acc[MTW][8];
  float m_run[MTW], l_run[MTW];
#pragma unroll
  for (int qt = 0; qt < MTW; ++qt) {
    // (finite: with -inf a masked score of the first step, -inf + inf, would hide from the test of the sum)
    m_run[qt] = -3.402823466e38f;
    l_run[qt] = 0.f;
#pragma unroll
    for (int ct = 0; ct < 8; ++ct) acc[qt][ct] = f32x4{0.f, 0.f, 0.f, 0.f};
  }

  const int k_rd = (8 * (i >> 2) + (i & 3)) * 256;
  const int v_rd = 2 * kBlockTok * kD + (j >> 1) * 4096 + (((2 * i + (j & 1)) ^ ((i >> 2) & 1)) << 4);
  auto run = [&](auto nt_tag) {
    constexpr int NTraw = decltype(nt_tag)::value;
    constexpr int NT = NTraw > 0 ? NTraw : 1;   // (no zero-length arrays; a wave without tiles only moves data)
    u32x4 kr[2][4], vr[8];
    auto read_k = [&](uint32_t ring) {
#pragma unroll
      for (int T = 0; T < 2; ++T)
#pragma unroll
        for (int kk = 0; kk < 4; ++kk)
          kr[T][kk] = *reinterpret_cast<const u32x4*>(lds.buf[0] + ring + k_rd + T * 4 * 256 + (((4 * kk + j) ^ i) << 4));
    };
    // slot 0 has landed when at most the two younger slots' loads are in flight
    __builtin_amdgcn_s_waitcnt(waitcnt_imm(2 * kLoads, 15));
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    if constexpr (NTraw > 0) read_k(0);
    uint32_t ring = 0;
    auto iteration = [&](auto last_tag, int n) {
      constexpr bool kLast = decltype(last_tag)::value;
      __builtin_amdgcn_s_waitcnt(waitcnt_imm(kLoads, 15));   // slot n+1 has landed
      asm volatile("" ::: "memory");
      __builtin_amdgcn_s_barrier();                          // ... for every wave; all have read V(n-1)
      asm volatile("" ::: "memory");
      issue((ring + 3 * kStepBytes) & (kRingBytes - 1));
      if constexpr (NTraw == 0) fetch_ids(n + 4);
      if constexpr (NTraw > 0) {
#pragma unroll
        for (int ct = 0; ct < 8; ++ct) vr[ct] = *reinterpret_cast<const u32x4*>(lds.buf[0] + ring + v_rd + ct * (16 * kPage * 2));
        f32x4 s[NT][2];
#pragma unroll
        for (int qt = 0; qt < NT; ++qt) s[qt][0] = s[qt][1] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kk = 0; kk < 4; ++kk)
#pragma unroll
          for (int qt = 0; qt < NT; ++qt) {
            s[qt][0] = mfma_16x16x32(kr[0][kk], qreg[qt][kk], s[qt][0]);
            s[qt][1] = mfma_16x16x32(kr[1][kk], qreg[qt][kk], s[qt][1]);
          }
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (!kLast) read_k((ring + kStepBytes) & (kRingBytes - 1));
        fetch_ids(n + 4);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (kLast) {
          const int t0 = tok_begin + n * kBlockTok;
          if (t0 + kBlockTok > tok_end) {   // wave-uniform: the ragged end of the chunk
#pragma unroll
            for (int qt = 0; qt < NT; ++qt)
#pragma unroll
              for (int e = 0; e < 4; ++e) {
                if (t0 + 8 * j + e >= tok_end) s[qt][0][e] = -INFINITY;
                if (t0 + 8 * j + 4 + e >= tok_end) s[qt][1][e] = -INFINITY;
              }
            // value slots no token owns may hold anything (NaN included): zero them
#pragma unroll
            for (int d = 0; d < 4; ++d) {
              const int tok = t0 + 8 * j + 2 * d;
              const uint32_t mask = (tok < tok_end ? 0x0000ffffu : 0u) | (tok + 1 < tok_end ? 0xffff0000u : 0u);
#pragma unroll
              for (int ct = 0; ct < 8; ++ct) vr[ct][d] &= mask;
            }
          }
        }
#pragma unroll
        for (int qt = 0; qt < NT; ++qt) {
          u32x4 pb;
          float psum;
          auto weights = [&] {
            float p[8];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              p[e] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[qt][0][e], sc, -m_run[qt]));
              p[4 + e] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[qt][1][e], sc, -m_run[qt]));
            }
            pb = u32x4{pack_bf16(p[0], p[1]), pack_bf16(p[2], p[3]), pack_bf16(p[4], p[5]), pack_bf16(p[6], p[7])};
            // (256-row blocks: the rounded weights, the same that multiply V)
            if constexpr (kHalves) psum = sum_bf16(pb);
            else psum = ((p[0] + p[1]) + (p[2] + p[3])) + ((p[4] + p[5]) + (p[6] + p[7]));
          };
          auto move_reference = [&] {
            const f32x4 s0 = s[qt][0], s1 = s[qt][1];
            const float mx = fmaxf(fmaxf(fmaxf(s0[0], s0[1]), fmaxf(s0[2], s0[3])),
                                   fmaxf(fmaxf(s1[0], s1[1]), fmaxf(s1[2], s1[3])));   // this lane's 8 tokens
            const float m_new = fmaxf(m_run[qt], rows_allreduce_max(mx) * sc);
            if (kHalves || __builtin_amdgcn_ballot_w64(m_new > m_run[qt]) != 0) {      // wave-uniform
              const float alpha = __builtin_amdgcn_exp2f(m_run[qt] - m_new);           // 1 where the row did not move
              l_run[qt] *= alpha;
              m_run[qt] = m_new;
#pragma unroll
              for (int ct = 0; ct < 8; ++ct) acc[qt][ct] *= alpha;
            }
          };
          if constexpr (kHalves) {
            weights();
            if (__builtin_amdgcn_ballot_w64(psum > kMaxWeight) != 0) {   // wave-uniform
              move_reference();
              weights();
            }
          } else {
            move_reference();
            weights();
          }
          l_run[qt] += psum;
#pragma unroll
          for (int ct = 0; ct < 8; ++ct) acc[qt][ct] = mfma_16x16x32(vr[ct], pb, acc[qt][ct]);
        }
      }
      ring = (ring + kStepBytes) & (kRingBytes - 1);
    };
    int n = 0;
    for (; n + 1 < nsteps; ++n) iteration(std::false_type{}, n);
    iteration(std::true_type{}, n);
  };
  if (nt == 2) run(std::integral_constant<int, 2>{});
  else if (nt == 1) run(std::integral_constant<int, 1>{});
  else run(std::integral_constant<int, 0>{});
  if (id_max >= (uint32_t)a.num_pages) bad_page = 1;

#pragma unroll
  for (int qt = 0; qt < MTW; ++qt) {
    const float l = rows_allreduce_sum(l_run[qt]);
    if (row_index[qt] >= 0) {
      const size_t ps = (size_t)row_index[qt] * nslot + slot;
      float* dst = a.partial_o + ps * kD + 4 * j;
#pragma unroll
      for (int ct = 0; ct < 8; ++ct) *reinterpret_cast<f32x4*>(dst + 16 * ct) = acc[qt][ct];
      if (j == 0) a.partial_ml[ps] = make_float2(m_run[qt], l);
    }
  }
  // the slots requested past the end write to LDS: the next item, or the end of the kernel, comes after
  __builtin_amdgcn_s_waitcnt(waitcnt_imm(0, 15));
  __syncthreads();
}

// Two shapes: blocks of 128 query rows, or, for groups with more than 128 rows, blocks of 256 rows whose
// halves are taken separately; both with workgroups of 4 waves, two per CU.
template <bool kWide>
__device__ __forceinline__ void prefix_kernel_body(const AttnArgs& a) {
  __shared__ PrefixLds lds;
  __shared__ int next_item;
  const int n_work = a.counters[MARL_CTR_NUM_PREFIX_ITEMS] * a.Hkv;
  // wide: entries of the queue come in groups of 16, the first halves of eight (item, KV head) pairs and
  // their second halves: workgroups are dealt to the eight XCDs in turn, so the halves of a pair meet
  // on one of them
  const int n_queue = kWide ? (n_work + 7) / 8 * 16 : n_work;
  int bad_page = 0;
  // The short suffix items go first: each round is a chain of dependent memory accesses with
  // little data, which is cheap while every workgroup has other work to overlap it with and
  // expensive at the tail of a kernel, where only a few workgroups are left.
  // (skipped when the plan found no such item: the scan of the short entries is a chain of
  // dependent loads at the very start of the kernel)
  if (a.counters[MARL_CTR_NUM_SHORT_PARTIAL_ITEMS] > 0) short_suffix_items<false>(a, bad_page);
  __syncthreads();
  for (bool first = true;; first = false) {   // first item = block index, as in the suffix kernel
    int qi = blockIdx.x;
    if (!first) {
      if (n_queue <= (int)gridDim.x) break;   // every entry has a workgroup of its own: no draw (hundreds of atomics on one word)
      if (threadIdx.x == 0) next_item = gridDim.x + atomicAdd(&a.counters[MARL_CTR_PREFIX_CURSOR], 1);
      __syncthreads();
      qi = next_item;
      __syncthreads();
    }
    if (qi >= n_queue) break;
    if constexpr (kWide) {
      const int pair = (qi >> 4) * 8 + (qi & 7);
      if (pair >= n_work) continue;           // workgroup-uniform
      const int4 it = a.prefix_items[pair / a.Hkv];
      prefix_item<true>(a, it, pair % a.Hkv, (qi >> 3) & 1, lds, bad_page);
    } else {
      const int4 it = a.prefix_items[qi / a.Hkv];
      prefix_item<false>(a, it, qi % a.Hkv, 0, lds, bad_page);
    }
  }
  if (bad_page) atomicOr(&a.counters[MARL_CTR_FLAGS], MARL_FLAG_BAD_PAGE);
}

__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2)))
void prefix_kernel(AttnArgs a) { prefix_kernel_body<false>(a); }
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2)))
void prefix_kernel_wide(AttnArgs a) { prefix_kernel_body<true>(a); }

// ---------------------------------------------------------------------------------------
// Items kernel: prefix and suffix items of calls of up to kOneQueueItems (sequence, KV head) pairs in one launch.
// Apart, the two kernels leave most of the GPU idle while the last items of the one and the first loads of
// the other are on their way; together they fill each other's gaps: 64 sequences in 4 groups, 64 / 8 heads, 512-2048 + about
// 1200 tokens: 25 + 54 us apart, 56 us in one.  Mean gain over 1371 random batches by the call's time: 15 % below 100 us,
// 13 % to 200, 6 % to 400.  From about 6144 pairs on there are enough items to fill the GPU, and the suffix kernel's
// three workgroups per CU (here two, for the prefix items' registers and LDS) are the better use of it: 1002 us apart and
// 1038 here for 2048 sequences x 4 KV heads, mean of that size 1.03, above 16384 0.96.
// One queue: the head of the suffix list, then the prefix items, then the other suffix items, so that the items that take
// longest come first (a prefix token keeps a workgroup busy about four times as long as a token of a suffix
// item, whose steps the waves share; the plan counts the head by that).  A sequence's suffix item may be done before
// the group's prefix partials are, so it is always left as a partial (but for sequences without a prefix) and the
// merge kernel adds them.  (Row tiles of the prefix as further suffix-like items, without the LDS ring: 88 instead of
// 72 us for the attention of the batch above, up to three times the time where groups are large.  Two steps in
// flight per wave, for which there are registers: 2-3 % slower, by batches of short items.)
// ---------------------------------------------------------------------------------------
template <bool kWide>
__device__ __forceinline__ void items_kernel_body(const AttnArgs& a) {
  __shared__ union { PrefixLds ring; ItemLds<1> item; } lds;
  __shared__ int next_item;
  const int n_long = a.counters[MARL_CTR_NUM_LONG_SUFFIX_ITEMS] * a.Hkv;
  const int pairs = a.counters[MARL_CTR_NUM_PREFIX_ITEMS] * a.Hkv;
  const int n_prefix = kWide ? (pairs + 7) / 8 * 16 : pairs;   // (halves of a wide block meet on an XCD, as in prefix_kernel_body)
  // Short items become partials only where their sequence has several chunks (the merge kernel takes the others).  In short
  // lists they are entries of the queue, else the waves take them first: drawn one by one they cost a draw each, and
  // so do those that are left to the merge kernel (1760 pairs of up to 283 tokens, 46.7 us apart: 60.4, now 46.4; 512
  // sequences of up to 1024 in chunks of 64, 28 / 4 heads, 273 apart: 404, now 268; by waves in short lists: 17.4 -> 23.1 for 117
  // pairs).  One draw per workgroup is about where the two meet: lists of 640 to 800 entries 4 % apart, either way.
  const bool partials = a.counters[MARL_CTR_NUM_SHORT_PARTIAL_ITEMS] > 0;
  const int n_all = a.counters[MARL_CTR_NUM_SUFFIX_ITEMS] * a.Hkv;
  const bool as_entries = partials && n_prefix + n_all <= (int)(gridDim.x + gridDim.x / 2);
  const int n_suffix = as_entries ? n_all : n_long;
  const int head = a.counters[MARL_CTR_NUM_FIRST_SUFFIX_ITEMS] * a.Hkv;
  const int i = threadIdx.x & 15;
  int bad_page = 0;
  if (partials && !as_entries) short_suffix_items<false>(a, bad_page);
  for (int e = blockIdx.x; e < n_prefix + n_suffix;) {   // workgroup-uniform
    if (e >= head && e < head + n_prefix) {
      const int qi = e - head;
      if constexpr (kWide) {
        const int pair = (qi >> 4) * 8 + (qi & 7);
        if (pair < pairs) prefix_item<true>(a, a.prefix_items[pair / a.Hkv], pair % a.Hkv, (qi >> 3) & 1, lds.ring, bad_page);
      } else {
        prefix_item<false>(a, a.prefix_items[qi / a.Hkv], qi % a.Hkv, 0, lds.ring, bad_page);
      }
    } else {
      const int qi = e < head ? e : e - n_prefix;
      const int4 it = a.suffix_items[qi / a.Hkv];
      const int kvh = qi % a.Hkv;
      const int s = it.x;
      const int row_index[1] = {i < a.R ? s * a.Hq + kvh * a.R + i : -1};
      const int chunks = ld_uniform(a.seq_chunks + s);
      if (qi < n_long || chunks >> 16 != 1)
        process_item<1, kSuffixWaves>(a, a.suffix_table + (size_t)s * a.max_sp, it.y, it.z, kvh, row_index,
                                      a.NCp + it.y / a.Cs, lds.item, bad_page, chunks == 1 << 16, 0);
    }
    if (n_prefix + n_suffix <= (int)gridDim.x) break;   // every item has a workgroup of its own
    if (threadIdx.x == 0) next_item = gridDim.x + atomicAdd(&a.counters[MARL_CTR_SUFFIX_CURSOR], 1);
    __syncthreads();
    e = next_item;
    __syncthreads();
  }
  if (bad_page) atomicOr(&a.counters[MARL_CTR_FLAGS], MARL_FLAG_BAD_PAGE);
}

static_assert(kSuffixWaves == 4, "prefix and suffix items share workgroups");
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2)))
void items_kernel(AttnArgs a) { items_kernel_body<false>(a); }
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2)))
void items_kernel_wide(AttnArgs a) { items_kernel_body<true>(a); }

// ---------------------------------------------------------------------------------------
// Merge kernel: the second reduction of split-KV decode attention.  For every (sequence,
// query head) it combines the partials of the group's prefix chunks and of the sequence's
// own suffix chunks, in slot order (so the sum order never changes between runs):
//   m* = max_i m_i,  out = sum_i O_i 2^(m_i - m*) / sum_i l_i 2^(m_i - m*)
// (m in log2 units).  A row without any token gives zeros.  Rows of a sequence whose own tokens
// are a single item are written where that item is processed (the suffix kernel, or this
// kernel's first phase for short items) and are not touched by the row loop.
//
// The kernel is a chain of dependent loads with almost no arithmetic, so it is organised to
// keep that chain short: the plan kernel has already stored each sequence's chunk counts
// (one load instead of group id -> prefix length), half a wave handles one row with 16-byte
// loads, and the first four partials of a row (max/sum and output) are all requested before
// any of them is used, as are the further ones, four at a time (their maxima eight at a time).  Every lane recomputes the few
// scalar weights itself: no shuffles.  (Further ones one after the other: 64 sequences with up to 13 partials a row, 64 / 8 heads,
// 71.8 us for the call instead of 70.0; 82 with up to 12, 28 / 4 heads, 55.1 and 53.1.)
// ---------------------------------------------------------------------------------------
constexpr int kMergeThreads = 256;
constexpr int kRowsPerBlock = kMergeThreads / 32;
constexpr int kEager = 4;   // partials fetched up front

__global__ __launch_bounds__(kMergeThreads) __attribute__((amdgpu_waves_per_eu(3, 3)))
void merge_kernel(AttnArgs a) {
  // (the row's chunk counts are requested before the short items: most workgroups have none of these, and
  // where every row is finished with them a workgroup is one load long instead of two)
  const int row = blockIdx.x * kRowsPerBlock + (threadIdx.x >> 5);
  const int info = row < a.NS * a.Hq ? a.seq_chunks[row / a.Hq] : 0x10000;
  const int own = a.one_queue && row < a.NS * a.Hq ? min(a.suffix_lens[row / a.Hq], a.max_sp * kPage) : 0;
  // first the sequences whose own tokens are one short item: attention over those tokens and
  // the merge with the group's prefix partials in one go, one item per wave
  {
    int bad_page = 0;
    short_suffix_items<true>(a, bad_page);
    if (bad_page) atomicOr(&a.counters[MARL_CTR_FLAGS], MARL_FLAG_BAD_PAGE);
  }
  const int sub = threadIdx.x & 31;   // lane within the half wave: channels 4*sub .. 4*sub+3
  const int npc = info & 0xffff, nsc = info >> 16;
  // a sequence whose own tokens are one item was finished where that item was processed: above
  // (at most kShortTokens tokens) or in the suffix kernel; the items kernel finishes only those without a prefix
  if (nsc == 1 && (npc == 0 || own <= kShortTokens)) return;
  const int n = npc + nsc;
  const int nslot = a.NCp + a.NCs;
  const float2* ml = a.partial_ml + (size_t)row * nslot;
  const float* po = a.partial_o + (size_t)row * nslot * kD + 4 * sub;
  auto slot_of = [&](int k) { return k < npc ? k : a.NCp + (k - npc); };

  float2 mlk[kEager];
  f32x4 ok[kEager];
#pragma unroll
  for (int k = 0; k < kEager; ++k) {
    mlk[k] = make_float2(-INFINITY, 0.f);
    ok[k] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (k < n) {
      const int sl = slot_of(k);
      mlk[k] = ml[sl];
      ok[k] = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(po + (size_t)sl * kD));
    }
  }
  float mstar = -INFINITY;
#pragma unroll
  for (int k = 0; k < kEager; ++k) mstar = fmaxf(mstar, mlk[k].x);
  for (int k = kEager; k < n; k += kMaximaAtOnce) {
    float mk[kMaximaAtOnce];
#pragma unroll
    for (int u = 0; u < kMaximaAtOnce; ++u) mk[u] = ml[slot_of(min(k + u, n - 1))].x;
#pragma unroll
    for (int u = 0; u < kMaximaAtOnce; ++u) mstar = fmaxf(mstar, mk[u]);
  }

  float denom = 0.f;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int k = 0; k < kEager; ++k) {
    const float f = (mlk[k].x == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(mlk[k].x - mstar);
    denom = __builtin_fmaf(mlk[k].y, f, denom);
    acc += ok[k] * f;
  }
  for (int k = kEager; k < n; k += kEager) {   // as many at once as before the first use
#pragma unroll
    for (int u = 0; u < kEager; ++u) {
      const int sl = slot_of(min(k + u, n - 1));
      mlk[u] = ml[sl];
      ok[u] = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(po + (size_t)sl * kD));
    }
#pragma unroll
    for (int u = 0; u < kEager; ++u) {
      const float f = (mlk[u].x == -INFINITY || k + u >= n) ? 0.f : __builtin_amdgcn_exp2f(mlk[u].x - mstar);
      denom = __builtin_fmaf(mlk[u].y, f, denom);
      acc += ok[u] * f;
    }
  }
  f32x4 r = {0.f, 0.f, 0.f, 0.f};
  if (n > 0 && denom > 0.f) r = acc * (1.0f / denom);
  if (a.out_dtype == MARL_OUT_F32) {
    *reinterpret_cast<f32x4*>(reinterpret_cast<float*>(a.out) + (size_t)row * kD + 4 * sub) = r;
  } else {
    typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
    const bf16x4 v = {(__bf16)r[0], (__bf16)r[1], (__bf16)r[2], (__bf16)r[3]};
    *reinterpret_cast<bf16x4*>(reinterpret_cast<uint16_t*>(a.out) + (size_t)row * kD + 4 * sub) = v;
  }
}

}  // namespace

int prefix_blocks_per_cu(bool wide) {
  int n = 0;
  const hipError_t e = wide ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, prefix_kernel_wide, 256, 0)
                            : hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, prefix_kernel, 256, 0);
  if (e != hipSuccess || n < 1) n = 1;
  return n;
}
int items_blocks_per_cu(bool wide) {
  int n = 0;
  const hipError_t e = wide ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, items_kernel_wide, 256, 0)
                            : hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, items_kernel, 256, 0);
  if (e != hipSuccess || n < 1) n = 1;
  return n;
}
int suffix_blocks_per_cu() {
  int n = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, suffix_kernel, kSuffixWaves * 64, 0) != hipSuccess || n < 1) n = 1;
  return n;
}

hipError_t launch_prefix(const AttnArgs& a, int grid, hipStream_t st) {
  if (a.qblock_rows == 256) hipLaunchKernelGGL(prefix_kernel_wide, dim3(grid), dim3(256), 0, st, a);
  else hipLaunchKernelGGL(prefix_kernel, dim3(grid), dim3(256), 0, st, a);
  return hipGetLastError();
}
hipError_t launch_suffix(const AttnArgs& a, int grid, hipStream_t st) {
  hipLaunchKernelGGL(suffix_kernel, dim3(grid), dim3(kSuffixWaves * 64), 0, st, a);
  return hipGetLastError();
}
hipError_t launch_items(const AttnArgs& a, int grid, hipStream_t st) {
  if (a.qblock_rows == kRowsPerQBlockWide) hipLaunchKernelGGL(items_kernel_wide, dim3(grid), dim3(256), 0, st, a);
  else hipLaunchKernelGGL(items_kernel, dim3(grid), dim3(256), 0, st, a);
  return hipGetLastError();
}
hipError_t launch_merge(const AttnArgs& a, hipStream_t st) {
  const long rows = (long)a.NS * a.Hq;
  if (rows == 0) return hipSuccess;
  // (a wave for every short item: with one head per KV head there are more of those than waves of rows, and a wave took two,
  // one after the other: 209 sequences of up to 76 tokens, 4 / 4 heads, 48.2 us for the call, now 41.1)
  const long grid = std::max((rows + kRowsPerBlock - 1) / kRowsPerBlock, ((long)a.NS * a.Hkv + kWaves - 1) / kWaves);
  hipLaunchKernelGGL(merge_kernel, dim3((unsigned)grid), dim3(kMergeThreads), 0, st, a);
  return hipGetLastError();
}

}  // namespace marl
