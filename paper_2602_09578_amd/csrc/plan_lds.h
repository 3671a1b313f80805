// The plan of a decode-attention call (group -> sequences CSR, the two work lists) built by one workgroup with its
// bookkeeping in LDS: device code shared by the plan kernels and by the kernel that serves a small call alone.
#ifndef MARL_PLAN_LDS_H
#define MARL_PLAN_LDS_H
#include <type_traits>

#include "marl_internal.h"
#include "wave_ops.h"

namespace marl {
namespace {

__device__ __forceinline__ int lane_id() { return threadIdx.x & 63; }
__device__ __forceinline__ int wave_id() { return threadIdx.x >> 6; }

__device__ __forceinline__ int wave_sum(int v) {
  return wave_allreduce(v, [](int x, int y) { return x + y; });
}

__device__ __forceinline__ int clamp_len(int v, int hi, int& flags) {
  const int c = min(max(v, 0), hi);
  if (c != v) flags |= MARL_FLAG_LEN_CLAMPED;
  return c;
}

// ---------------------------------------------------------------------------------------
// The plan of plan_kernel.hip for shapes whose bookkeeping fits in LDS (sizes below, chunks <= 8192
// tokens): inputs are read once into registers, counts, offsets, member lists and histograms
// live in LDS, and global memory only sees the final stores.  The general plan kernel pays
// a chain of ~30 dependent global round trips; this one pays one.  What bounds it is the chain of
// barriers and LDS round trips of its one workgroup: the three scans (groups, suffix and prefix classes)
// share one pass and stay in the vector ALU.  16 sequences 9.9 -> 7.2 us, 2048 sequences 12.0 -> 9.9 us, launch
// included; the former time had a block-wide scan with shuffles and three barriers for each of the three.  (One LDS atomic
// for all lanes of a wave that count in the same word: 11.9 -> 16.5 us, 2048 sequences; 14.4 -> 23.6, 4096.  But whole chunks, which
// are all of one class, take their places by one atomic per wave: lanes that add to the same word one after the other, and
// wait for what they get, took 4 us of the plan of 256 sequences of several chunks, 10.7 -> 6.5 us as a replayed graph, 1 us for
// 64 sequences, 6.7 -> 5.6, both with the code for two sequences per thread.  With eight or 32 per thread, whose scans run
// whether there are whole chunks or not, 14.4 -> 15.2 us for 8000 sequences, 42 -> 52 for 20000: an atomic each there.)
// ---------------------------------------------------------------------------------------
// Four sizes: up to 512 sequences and groups by 256 threads, beside a small call's attention (13 KB of LDS); up to 2048
// sequences in 1024 groups (22 KB), up to 8192 in 2048 (56 KB) and up to 32768 sequences in 8192 groups with 16-bit member ids (130 KB of the 160 KB), by
// 1024 threads.
constexpr int kSmallMaxClasses = 256;

// kCheckPages: the plan's workgroup also looks for block-table entries outside the pool among those of addressed
// tokens (where nobody else reports them).
template <int kThreads, int kSmallMaxSeqs, int kSmallMaxGroups, class MemberId, bool kCheckPages = false>
__device__ __forceinline__ void plan_in_lds(const AttnArgs& a) {
  constexpr int kSeqsPerThread = kSmallMaxSeqs / kThreads;
  constexpr int kGroupsPerThread = kSmallMaxGroups / kThreads;
  __shared__ int cnt[kSmallMaxGroups];
  __shared__ int start[kSmallMaxGroups];
  __shared__ MemberId members[kSmallMaxSeqs];
  __shared__ int hist_s[kSmallMaxClasses];
  __shared__ int hist_p[kSmallMaxClasses];
  __shared__ int tmp[kThreads / 64];
  __shared__ int n_long_items, n_short_partial_items, n_suffix_items, n_prefix_items;
  // clamped prefix lengths, where there is room for them (else they are re-read from global memory)
  constexpr bool kPrefixLensInLds = kSmallMaxGroups <= 2048;
  __shared__ int prefix_len[kPrefixLensInLds ? kSmallMaxGroups : 1];
  const int tid = threadIdx.x;
  const int Cs = a.Cs, Cp = a.Cp, R = a.R, QB = a.qblock_rows;
  const int max_st = a.max_sp * kPage, max_pt = a.max_pp * kPage;
  int flags = 0;

  // inputs -> registers (the only loads from global memory).  The larger size has no room for
  // 3 x 32 values per thread: it keeps only the ranks and re-reads group ids and lengths (cache
  // hits) in the later phases.
  constexpr bool kKeep = kSeqsPerThread <= 8;
  int g_keep[kKeep ? kSeqsPerThread : 1], S_keep[kKeep ? kSeqsPerThread : 1], rank_of[kSeqsPerThread];
  if constexpr (kKeep) {
#pragma unroll
    for (int k = 0; k < kSeqsPerThread; ++k) {
      const int s = tid + k * kThreads;
      g_keep[k] = s < a.NS ? a.group_of_seq[s] : -1;
      S_keep[k] = s < a.NS ? a.suffix_lens[s] : 0;
    }
  }
  int ignored = 0;
  auto G = [&](int k) {   // group id of this thread's k-th sequence (only called for s < NS)
    if constexpr (kKeep) return g_keep[k]; else return a.group_of_seq[tid + k * kThreads];
  };
  auto S_len = [&](int k) {   // its clamped suffix length
    if constexpr (kKeep) return S_keep[k]; else return clamp_len(a.suffix_lens[tid + k * kThreads], max_st, ignored);
  };
  int P_of[kGroupsPerThread];
#pragma unroll
  for (int k = 0; k < kGroupsPerThread; ++k) {
    const int g = tid + k * kThreads;
    P_of[k] = g < a.NG ? a.prefix_lens[g] : 0;
  }
  for (int i = tid; i < kSmallMaxGroups; i += kThreads) cnt[i] = 0;
  for (int i = tid; i < kSmallMaxClasses; i += kThreads) { hist_s[i] = 0; hist_p[i] = 0; }
  __shared__ int longest_prefix, any_ranked;
  if (tid == 0) { n_long_items = 0; n_short_partial_items = 0; longest_prefix = 0; any_ranked = 0; }
  if (tid < 64) a.counters[tid] = 0;
  __syncthreads();

  // full chunks and long items are counted per thread and added once per wave: nearly every
  // sequence contributes to these two words, and same-address LDS atomics run one lane at a time
  int nfull_mine = 0, nlong_mine = 0, nshort_partial_mine = 0;
#pragma unroll
  for (int k = 0; k < kSeqsPerThread; ++k) {
    const int s = tid + k * kThreads;
    rank_of[k] = -1;
    if (s < a.NS) {
      const int g = G(k);
      if ((unsigned)g < (unsigned)a.NG) rank_of[k] = atomicAdd(&cnt[g], 1);
      else flags |= MARL_FLAG_BAD_GROUP;
      int S;
      if constexpr (kKeep) S = S_keep[k] = clamp_len(S_keep[k], max_st, flags);
      else S = clamp_len(a.suffix_lens[s], max_st, flags);
      const int nfull = S / Cs, tail = S % Cs;
      nfull_mine += nfull;
      if (tail) atomicAdd(&hist_s[(Cs - tail) / 32], 1);
      nlong_mine += (Cs > kShortTokens ? nfull : 0) + (tail > kShortTokens ? 1 : 0);
    // short items (at most kShortTokens tokens) of sequences with several suffix chunks: they become partials
    if (nfull + (tail > 0) >= 2)
      nshort_partial_mine += (Cs <= kShortTokens ? nfull : 0) + ((tail > 0 && tail <= kShortTokens) ? 1 : 0);
    }
  }
  nfull_mine = wave_sum(nfull_mine);
  nlong_mine = wave_sum(nlong_mine);
  nshort_partial_mine = wave_sum(nshort_partial_mine);
  if (lane_id() == 0) {
    if (nfull_mine) atomicAdd(&hist_s[0], nfull_mine);
    if (nlong_mine) atomicAdd(&n_long_items, nlong_mine);
    if (nshort_partial_mine) atomicAdd(&n_short_partial_items, nshort_partial_mine);
  }
  __syncthreads();

  int longest = 0;
  // prefix items by class; the counts' sums inside a wave (thread t: groups kGroupsPerThread t ..)
#pragma unroll
  for (int k = 0; k < kGroupsPerThread; ++k) {
    const int g = tid + k * kThreads;
    if (g < a.NG) {
      P_of[k] = clamp_len(P_of[k], max_pt, flags);
      if constexpr (kPrefixLensInLds) prefix_len[g] = P_of[k];
      const int nqb = (cnt[g] * R + QB - 1) / QB;
      const int nfull = P_of[k] / Cp, tail = P_of[k] % Cp;
      if (nqb) {
        if (nfull) atomicAdd(&hist_p[0], nfull * nqb);
        if (tail) atomicAdd(&hist_p[(Cp - tail) / 32], nqb);
        longest = max(longest, min(P_of[k], Cp));
      }
    }
  }
  // (one atomic per wave: one per group took 1.7 us of the plan of 256 groups)
  longest = wave_allreduce(longest, [](int x, int y) { return max(x, y); });
  if (lane_id() == 0 && longest > 0) atomicMax(&longest_prefix, longest);
  int own = 0;
#pragma unroll
  for (int k = 0; k < kGroupsPerThread; ++k) own += cnt[tid * kGroupsPerThread + k];   // (zero from NG on)
  const int own_end = wave_inclusive_scan(own);
  if (lane_id() == 63) tmp[wave_id()] = own_end;
  __syncthreads();

  // starts of the groups, of the suffix classes (wave 0) and of the prefix classes (wave 1); afterwards
  // the histograms serve as per-class cursors
  constexpr int kPlanWaves = kThreads / 64;
  const int upto = wave_inclusive_scan(lane_id() < kPlanWaves ? tmp[lane_id()] : 0);
  const int nseq_grouped = __builtin_amdgcn_readlane(upto, kPlanWaves - 1);
  const int wave_s = __builtin_amdgcn_readfirstlane(wave_id());
  int at = own_end - own + (wave_s > 0 ? __builtin_amdgcn_readlane(upto, wave_s - 1) : 0);
#pragma unroll
  for (int k = 0; k < kGroupsPerThread; ++k) {
    start[tid * kGroupsPerThread + k] = at;
    at += cnt[tid * kGroupsPerThread + k];
  }
  if (wave_s < 2) {
    constexpr int kPer = kSmallMaxClasses / 64;
    int* hist = (wave_s == 0 ? hist_s : hist_p) + lane_id() * kPer;
    int v[kPer], mine = 0;
#pragma unroll
    for (int k = 0; k < kPer; ++k) mine += v[k] = hist[k];   // (zero from the number of classes on)
    const int end = wave_inclusive_scan(mine);
    int first = end - mine;
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      hist[k] = first;
      first += v[k];
    }
    if (lane_id() == 63) (wave_s == 0 ? n_suffix_items : n_prefix_items) = end;
  }
  __syncthreads();

  // Whole chunks' places by one atomic per wave.  Whether a wave has any is known from the sums above: most small calls have
  // none, and a test in each round was 0.07 us of a call of 5.
  constexpr bool kTogether = kSeqsPerThread <= 2;
  const bool whole_s = __builtin_amdgcn_readfirstlane(nfull_mine) > 0, whole_p = __builtin_amdgcn_readfirstlane(longest) == Cp;
  auto take = [&](int* word, int n) {               // (for all lanes of the wave)
    const int inc = wave_inclusive_scan(n);
    int base = 0;
    if (lane_id() == 63) base = atomicAdd(word, inc);
    return __builtin_amdgcn_readlane(base, 63) + inc - n;
  };
  auto put_suffix = [&](int pos, int s, int nfull) {
    for (int i = 0; i < nfull; ++i) a.suffix_items[pos + i] = make_int4(s, i * Cs, (i + 1) * Cs, 0);
  };
  auto put_prefix = [&](int pos, int g, int nfull, int nqb) {
    for (int i = 0; i < nfull; ++i)
      for (int b = 0; b < nqb; ++b)
        a.prefix_items[pos + i * nqb + b] = make_int4(g, i * Cp, (i + 1) * Cp, b * QB);
  };
#pragma unroll
  for (int k = 0; k < kSeqsPerThread; ++k) {
    const int s = tid + k * kThreads;
    int nfull_of = 0;
    if (s < a.NS) {
      const int g = G(k);
      if (rank_of[k] >= 0) members[start[g] + rank_of[k]] = (MemberId)s;
      const int S = S_len(k);
      int P = 0;
      if (rank_of[k] >= 0) {
        int dummy = 0;
        if constexpr (kPrefixLensInLds) P = prefix_len[g];
        else P = clamp_len(a.prefix_lens[g], max_pt, dummy);
      }
      a.seq_chunks[s] = ((P + Cp - 1) / Cp) | (((S + Cs - 1) / Cs) << 16);
      const int nfull = S / Cs, tail = S % Cs;
      if constexpr (kTogether) nfull_of = nfull;
      else if (nfull) put_suffix(atomicAdd(&hist_s[0], nfull), s, nfull);
      if (tail) {
        const int pos = atomicAdd(&hist_s[(Cs - tail) / 32], 1);
        a.suffix_items[pos] = make_int4(s, nfull * Cs, S, 0);
      }
    }
    if constexpr (kTogether)
      if (whole_s && __builtin_amdgcn_ballot_w64(nfull_of > 0) != 0) put_suffix(take(&hist_s[0], nfull_of), s, nfull_of);   // wave-uniform
  }
  bool ranked = false;   // a group that has an order
#pragma unroll
  for (int k = 0; k < kGroupsPerThread; ++k) {
    const int g = tid + k * kThreads;
    int nfull_of = 0, nqb_of = 0;
    if (g < a.NG) {
      a.group_count[g] = cnt[g];
      ranked |= cnt[g] >= 2 && cnt[g] <= 64;
      a.group_start[g] = start[g];
      const int P = P_of[k];
      const int nqb = (cnt[g] * R + QB - 1) / QB;
      const int nfull = P / Cp, tail = P % Cp;
      if (nqb) {
        if constexpr (kTogether) nfull_of = nfull, nqb_of = nqb;
        else if (nfull) put_prefix(atomicAdd(&hist_p[0], nfull * nqb), g, nfull, nqb);
        if (tail) {
          const int pos = atomicAdd(&hist_p[(Cp - tail) / 32], nqb);
          for (int b = 0; b < nqb; ++b)
            a.prefix_items[pos + b] = make_int4(g, nfull * Cp, P, b * QB);
        }
      }
    }
    if constexpr (kTogether)
      if (whole_p && __builtin_amdgcn_ballot_w64(nfull_of > 0) != 0) put_prefix(take(&hist_p[0], nfull_of * nqb_of), g, nfull_of, nqb_of);
  }
  if (tid == 0) a.group_start[a.NG] = nseq_grouped;
  if (ranked) any_ranked = 1;
  __syncthreads();

  // ascending sequence id inside every group of at most 64 members (as in the general kernel).  Lanes of a wave usually get their
  // ranks in order, so a group whose members stand side by side is in order already: only one where a member finds
  // a later sequence before it is ranked by counting (launch included, 128 groups of 64: 52.6 -> 31 us, 64 of 32: 14.8 -> 12.6,
  // 20 of 64: 13.6 -> 10.8; 85 of 24, of which some lie in two waves: 13.0 and 12.9; none to order: the same).
  constexpr int kOutOfOrder = 1 << 30;
  if (any_ranked) {   // workgroup-uniform
#pragma unroll
    for (int k = 0; k < kSeqsPerThread; ++k) {
      const int s = tid + k * kThreads;
      if (s < a.NS && rank_of[k] > 0) {
        const int g = G(k);
        if ((int)members[start[g] + rank_of[k] - 1] > s) atomicOr(&cnt[g], kOutOfOrder);
      }
    }
    __syncthreads();
  }
#pragma unroll
  for (int k = 0; k < kSeqsPerThread; ++k) {
    const int s = tid + k * kThreads;
    if (s < a.NS && rank_of[k] >= 0) {
      const int g = G(k);
      const int b = start[g], n = cnt[g] & (kOutOfOrder - 1);
      int place = rank_of[k];
      if (n <= 64 && n != cnt[g]) {
        place = 0;
        for (int m0 = 0; m0 < n; m0 += 8) {   // (eight reads in flight)
          int v[8];
#pragma unroll
          for (int u = 0; u < 8; ++u) v[u] = (int)members[b + min(m0 + u, n - 1)];
#pragma unroll
          for (int u = 0; u < 8; ++u) place += m0 + u < n && v[u] < s;
        }
      }
      a.group_seqs[b + place] = s;
    }
  }
  if constexpr (kCheckPages) {
    static_assert(kPrefixLensInLds && kKeep, "lengths at hand");
    __shared__ int suffix_len[kSmallMaxSeqs];
#pragma unroll
    for (int k = 0; k < kSeqsPerThread; ++k)
      if (tid + k * kThreads < a.NS) suffix_len[tid + k * kThreads] = S_keep[k];
    __syncthreads();
    // Entries of addressed tokens only: tables of a fixed capacity are mostly padding, and looking through all of it took one
    // workgroup longer than the attention (one sequence of 40 tokens in a row for 2^20: 29.8 us, now 8.5, general kernels 14.7;
    // 512 of up to 40 in rows for 2048: 33.8, now 13.2, 23.4).  A power of two lanes share a row, as many as there are for each.
    // With at most a row for each team of lanes a lane requests sixteen of its entries together, else two of four rows (eight
    // instead of sixteen: 16 rows of 1024 entries 29.7 us, now 28.4; 16 bytes at a time, or four of four rows, or one of eight:
    // 512 rows of 3 entries 10.1 to 10.6 us, now 10.0).
    auto check = [&](const int32_t* table, const int rows, const int pages, auto&& tokens) {
      if (rows == 0 || pages == 0) return;   // workgroup-uniform, as all of the loops' bounds but the lengths
      int lanes = 8;
      while (2 * lanes * rows <= kThreads) lanes *= 2;
      const int teams = kThreads / lanes, team = tid / lanes, lane = tid & (lanes - 1);
      auto look = [&](auto rows_tag, auto entries_tag) {
        constexpr int kRows = decltype(rows_tag)::value, kPieces = decltype(entries_tag)::value;
        for (int r0 = team; r0 < rows; r0 += kRows * teams) {
          int n[kRows], longest = 0;
#pragma unroll
          for (int u = 0; u < kRows; ++u) {
            n[u] = r0 + u * teams < rows ? (tokens(r0 + u * teams) + kPage - 1) / kPage : 0;
            longest = max(longest, n[u]);
          }
          for (int p0 = lane; p0 < longest; p0 += kPieces * lanes) {
            int id[kRows][kPieces];
#pragma unroll
            for (int u = 0; u < kRows; ++u)
#pragma unroll
              for (int k = 0; k < kPieces; ++k)   // (in the row whatever its length)
                id[u][k] = table[(size_t)min(r0 + u * teams, rows - 1) * pages + max(min(p0 + k * lanes, n[u] - 1), 0)];
#pragma unroll
            for (int u = 0; u < kRows; ++u)
#pragma unroll
              for (int k = 0; k < kPieces; ++k)
                if ((unsigned)id[u][k] >= (unsigned)a.num_pages && n[u] > 0) flags |= MARL_FLAG_BAD_PAGE;   // (past the end: the last one again)
          }
        }
      };
      if (rows <= teams) look(std::integral_constant<int, 1>{}, std::integral_constant<int, 16>{});
      else look(std::integral_constant<int, 4>{}, std::integral_constant<int, 2>{});
    };
    check(a.suffix_table, a.NS, a.max_sp, [&](int s) { return suffix_len[s]; });
    check(a.prefix_table, a.NG, a.max_pp, [&](int g) { return cnt[g] ? prefix_len[g] : 0; });
  }
  if (flags) atomicOr(&a.counters[MARL_CTR_FLAGS], flags);
  if (tid == 0) {
    a.counters[MARL_CTR_NUM_SUFFIX_ITEMS] = n_suffix_items;
    a.counters[MARL_CTR_NUM_PREFIX_ITEMS] = n_prefix_items;
    a.counters[MARL_CTR_NUM_LONG_SUFFIX_ITEMS] = n_long_items;
    a.counters[MARL_CTR_NUM_SHORT_PARTIAL_ITEMS] = n_short_partial_items;
    const int len = longest_prefix * kPrefixTokenCost;
    a.counters[MARL_CTR_NUM_FIRST_SUFFIX_ITEMS] = len <= Cs && Cs > kShortTokens && longest_prefix > 0 ? hist_s[min((Cs - max(len, kShortTokens + 1)) / 32, kSmallMaxClasses - 1)] : 0;
  }
}

}  // namespace
}  // namespace marl
#endif  // MARL_PLAN_LDS_H
