// Sampling fused with the log-probability: one streaming pass over a row's logits yields
// what is needed to draw a token from softmax(logits / T) by inverse-CDF with a uniform
// number supplied by the caller, and that token's log-probability (rollout produces both for
// every generated token; the paper trains with GRPO, Section 8.1, which consumes the latter).
//
// Rows are taken whole by a workgroup each, or divided between workgroups (launch_sample), which takes two kernels.
// Pass 1 (streaming, the cost of the log-prob kernel): every wave takes contiguous chunks of
//   4096 logits and stores each chunk's (max, sum of 2^(y - max)), y = x * log2(e) / T.
// Pass 2 (one wave per row, re-reads 8 KB): an ordered scan over the chunk sums finds the chunk
//   in which the cumulative probability passes u, an ordered scan inside that chunk finds the
//   token.  Token = first t with sum_{v <= t} p_v > u; if rounding leaves none, the last token
//   with non-zero probability.  The running sums of a scan are associated differently from lane to
//   lane, so a lane without mass (masked tokens, positions past the end) can be the first whose sum
//   passes: only chunks, lanes and tokens that have mass are ever taken.
#include <algorithm>
#include <type_traits>

#include "marl_internal.h"
#include "wave_ops.h"

namespace marl {
namespace {

constexpr int kChunk = 4096;          // logits per wave chunk: 8 iterations x 64 lanes x 8
constexpr int kIters = kChunk / 512;
// A chunk of less mass than this, relative to the row's largest weight, holds no token that can be drawn: a sum of
// up to 4096 weights above it has one of at least 2^-124, which is not flushed to zero where weights are formed again.
constexpr double kLeastMass = 0x1p-112;
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef u32x4 u32x4_any __attribute__((aligned(2)));   // 16-byte access at any element (the GPU's global loads take any alignment)

__device__ __forceinline__ float ex2(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ __forceinline__ float ex2_diff(float a, float b) { return ex2(a - (b == -INFINITY ? 0.f : b)); }

// the 8 logits at x[pos .. pos+8) as four packed words (token 2d in the low half of word d);
// positions past the end read as -inf.  One 16-byte load when all 8 exist, at any alignment (rows of
// an odd vocabulary start anywhere).
__device__ __forceinline__ u32x4 load8_words(const uint16_t* x, long pos, long end) {
  const uint16_t* p = x + pos;
  if (pos + 8 <= end) return __builtin_nontemporal_load(reinterpret_cast<const u32x4_any*>(p));
  u32x4 v;
#pragma unroll
  for (int d = 0; d < 4; ++d) {
    const uint32_t lo = pos + 2 * d < end ? p[2 * d] : 0xff80u;
    const uint32_t hi = pos + 2 * d + 1 < end ? p[2 * d + 1] : 0xff80u;
    v[d] = lo | (hi << 16);
  }
  return v;
}

// Where a row ends, in two steps, so that loads stay in flight together: the 8 logits at x[pos .. pos+8) or, if the row ends before,
// its last 8 (end >= 8), and when they are used the shift that puts them in their places and -inf behind them.  (Element by element,
// in branches, the loads of a last chunk wait for each other, and most rows have one: 13 x 4099 6.74 -> 5.84 us, 250 x 32000 7.96 -> 6.98, 13 x
// 152064 9.3 -> 7.7, 2410 x 20481 33.5 -> 30.7.  The top-p kernel has no registers left for it: 2 to 7 % slower with it where it counts
// whole rows.)
__device__ __forceinline__ u32x4 load8_clamped(const uint16_t* x, long pos, long end) {
  return __builtin_nontemporal_load(reinterpret_cast<const u32x4_any*>(x + min(pos, end - 8)));
}
__device__ __forceinline__ u32x4 end_in_place(u32x4 v, long pos, long end) {
  const int s = (int)min(max(pos - (end - 8), 0l), 8l);   // logits of v that belong to the lanes before
  constexpr unsigned long long kNone = 0xff80ff80ff80ff80ull;
  unsigned long long lo = v[0] | (unsigned long long)v[1] << 32, hi = v[2] | (unsigned long long)v[3] << 32;
  if (s & 4) { lo = hi; hi = kNone; }
  const int r = (s & 3) * 16;
  lo = lo >> r | hi << (63 - r) << 1;
  hi = hi >> r | kNone << (63 - r) << 1;
  if (s == 8) lo = hi = kNone;
  return u32x4{(uint32_t)lo, (uint32_t)(lo >> 32), (uint32_t)hi, (uint32_t)(hi >> 32)};
}

template <class T>
__device__ __forceinline__ T wave_allreduce_sum(T v) { return wave_allreduce(v, [](T x, T y) { return x + y; }); }
__device__ __forceinline__ float wave_max(float v) { return wave_allreduce(v, [](float x, float y) { return fmaxf(x, y); }); }
__device__ __forceinline__ float wave_sum(float v) { return wave_allreduce_sum(v); }
// the value of one lane (wave-uniform index) in every lane, through a scalar register
__device__ __forceinline__ int from_lane(int v, int l) { return __builtin_amdgcn_readlane(v, l); }
__device__ __forceinline__ float from_lane(float v, int l) {
  return __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(v), l));
}
__device__ __forceinline__ double from_lane(double v, int l) {
  const unsigned long long u = __builtin_bit_cast(unsigned long long, v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)u, l);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), l);
  return __builtin_bit_cast(double, (unsigned long long)lo | ((unsigned long long)hi << 32));
}

// The logits of a chunk, as a wave holds them; requested, and as they are used.  (kAnyLength: also of a row of fewer than 8.)
template <bool kAnyLength = true>
__device__ __forceinline__ void fetch_chunk(const uint16_t* x, long base, int lane, long vocab, u32x4 (&w)[kIters]) {
  if (base + kChunk <= vocab) {   // wave-uniform
#pragma unroll
    for (int it = 0; it < kIters; ++it) w[it] = __builtin_nontemporal_load(reinterpret_cast<const u32x4_any*>(x + base + it * 512 + lane * 8));
  } else if (!kAnyLength || vocab >= 8) {
#pragma unroll
    for (int it = 0; it < kIters; ++it) w[it] = load8_clamped(x, base + it * 512 + lane * 8, vocab);
  } else {
#pragma unroll
    for (int it = 0; it < kIters; ++it) w[it] = load8_words(x, base + it * 512 + lane * 8, vocab);
  }
}
__device__ __forceinline__ void end_chunk(long base, int lane, long vocab, u32x4 (&w)[kIters]) {
  if (base + kChunk <= vocab || vocab < 8) return;   // wave-uniform
#pragma unroll
  for (int it = 0; it < kIters; ++it)
    if (base + (it + 1) * 512 > vocab) w[it] = end_in_place(w[it], base + it * 512 + lane * 8, vocab);
}
// (max, sum of 2^(y - max)) of a chunk.  Per lane a running (largest raw logit, sum relative to it), 16 logits at
// a time as they arrive: with the wave's maximum first, all of a batch's waves waited for whole chunks and then
// summed together.
__device__ __forceinline__ float2 chunk_sum(const u32x4 (&w)[kIters], float c) {
  float xr = -INFINITY, sr = 0.f;
#pragma unroll
  for (int it = 0; it < kIters; it += 2) {
    float xn = xr;
#pragma unroll
    for (int i = it; i < it + 2; ++i)
#pragma unroll
      for (int d = 0; d < 4; ++d)
        xn = fmaxf(xn, fmaxf(__uint_as_float(w[i][d] << 16), __uint_as_float(w[i][d] & 0xffff0000u)));
    const float ms = xn == -INFINITY ? 0.f : xn * c;   // c > 0: the scaled maximum is the maximum of the scaled values
    float s0 = 0.f, s1 = 0.f;
#pragma unroll
    for (int i = it; i < it + 2; ++i)
#pragma unroll
      for (int d = 0; d < 4; ++d) {
        s0 += ex2(__builtin_fmaf(__uint_as_float(w[i][d] << 16), c, -ms));
        s1 += ex2(__builtin_fmaf(__uint_as_float(w[i][d] & 0xffff0000u), c, -ms));
      }
    sr = sr * ex2(xr * c - ms) + (s0 + s1);
    xr = xn;
  }
  const float m = wave_max(xr) * c;
  return make_float2(m, wave_sum(sr * ex2_diff(xr * c, m)));
}

// grid: rows * groups_per_row workgroups of 4 waves; a workgroup covers 4 * chunks_per_wave
// consecutive chunks of one row, wave w taking chunks first + w, first + w + 4, ...
__global__ __launch_bounds__(256) void sample_scan_kernel(SampleArgs a) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int row = blockIdx.x / a.groups_per_row;
  const int first = (blockIdx.x % a.groups_per_row) * 4 * a.chunks_per_wave;
  const uint16_t* x = a.logits + (size_t)row * a.vocab;
  // the words of the wave's next chunk are requested before the current chunk is reduced
  // (rows of fewer than 8 chunks are not divided; with the loads of the shortest ones four registers more: 300 x 65537 14.7 us, now 14.3,
  // 600 x 28673 15.6 and 15.1)
  u32x4 cur[kIters], nxt[kIters];
  if (first + wave < a.num_chunks) fetch_chunk<false>(x, (long)(first + wave) * kChunk, lane, a.vocab, cur);
  for (int k = 0; k < a.chunks_per_wave; ++k) {
    const int chunk = first + wave + 4 * k;
    if (chunk >= a.num_chunks) break;
    const bool more = k + 1 < a.chunks_per_wave && chunk + 4 < a.num_chunks;   // wave-uniform
    if (more) fetch_chunk<false>(x, (long)(chunk + 4) * kChunk, lane, a.vocab, nxt);
    end_chunk((long)chunk * kChunk, lane, a.vocab, cur);
    const float2 v = chunk_sum(cur, a.inv_temp_log2e);
    if (lane == 0) a.partials[(size_t)row * a.num_chunks + chunk] = v;
    if (more) {
#pragma unroll
      for (int it = 0; it < kIters; ++it) cur[it] = nxt[it];
    }
  }
}

// Draws the row's token from its chunks' sums (global memory or LDS), one wave.  It is a chain of dependent
// reads (chunk sums, then the chosen chunk), so each of them is one round trip: the sums of the first 64 chunks (all of
// them up to a vocabulary of 262144) are read once and stay in a register, and the chunk's logits
// are requested together (256 rows x 152064: 10.5 us with the sums re-read for every use and the chunk in eight
// dependent pieces, 4.8 us as a kernel of its own).
__device__ __forceinline__ void pick_token(const SampleArgs& a, const float2* part, const int num_chunks, const int row, const float u) {
  const int lane = threadIdx.x & 63;
  const uint16_t* x = a.logits + (size_t)row * a.vocab;
  const float c = a.inv_temp_log2e;
  const float2 first = lane < num_chunks ? part[lane] : make_float2(-INFINITY, 0.f);
  auto chunk_sum = [&](int base) {   // (max, sum) of chunk base + lane
    if (base == 0) return first;
    return base + lane < num_chunks ? part[base + lane] : make_float2(-INFINITY, 0.f);
  };
  // global max and total, chunk sums rescaled to the global max.  The few dozen chunk sums are
  // accumulated in double precision: they decide in which chunk the uniform number falls, and a
  // float32 running sum over the whole vocabulary would move a CDF step by up to ~1e-5.
  float M = -INFINITY;
  for (int base = 0; base < num_chunks; base += 64) M = fmaxf(M, chunk_sum(base).x);
  M = wave_max(M);
  auto chunk_mass = [&](int base) -> double {
    const float2 p = chunk_sum(base);
    return base + lane < num_chunks ? (double)(p.y * ex2_diff(p.x, M)) : 0.0;
  };
  double total = 0.0;
  for (int base = 0; base < num_chunks; base += 64)   // fixed order: tiles of 64 chunks
    total += from_lane(wave_inclusive_scan(chunk_mass(base)), 63);
  const double target = (double)u * total;
  const double least = kLeastMass * fmin(total, 1.0);
  // the chunk in which the running sum passes the target
  double before = 0.0;
  bool take_last = false;
  int chunk = -1, last_nonzero = -1;
  for (int base = 0; base < num_chunks && chunk < 0; base += 64) {
    const double v = chunk_mass(base);
    const double cum = before + wave_inclusive_scan(v);
    const bool some = v > least;
    const unsigned long long hit = __builtin_amdgcn_ballot_w64(some && cum > target);
    const unsigned long long nz = __builtin_amdgcn_ballot_w64(some);
    if (nz) last_nonzero = base + 63 - __builtin_clzll(nz);
    if (hit) {
      const int l = __builtin_ctzll(hit);
      chunk = base + l;
      before = from_lane(cum - v, l);
    } else {
      before = from_lane(cum, 63);
    }
  }
  if (chunk < 0) {   // rounding: u * total not below the last partial sum
    chunk = max(last_nonzero, 0);
    take_last = true;   // any non-zero element of the chunk passes; the last one is taken below
  }
  // remaining mass to pass inside the chunk (inf: nothing passes, the last non-zero token is taken)
  const float want = take_last ? INFINITY : (float)(target - before);
  const long cbase = (long)chunk * kChunk + lane * 8;
  u32x4 words[kIters];
  fetch_chunk(x, (long)chunk * kChunk, lane, a.vocab, words);
  end_chunk((long)chunk * kChunk, lane, a.vocab, words);
  // the weights 2^(y - M) of 8 logits, the same each time they are formed
  const float ms = M == -INFINITY ? 0.f : M;
  auto weights = [&](u32x4 v, float (&w)[8]) {
    float s = 0.f;
#pragma unroll
    for (int d = 0; d < 4; ++d) {
      w[2 * d] = ex2(__builtin_fmaf(__uint_as_float(v[d] << 16), c, -ms));
      w[2 * d + 1] = ex2(__builtin_fmaf(__uint_as_float(v[d] & 0xffff0000u), c, -ms));
      s += w[2 * d];
      s += w[2 * d + 1];
    }
    return s;
  };
  // the piece of 512 tokens in which the running sum passes (`at`), else the last one with any mass
  float run = 0.f, cum_at = 0.f;
  int at = -1, last = -1;
#pragma unroll
  for (int it = 0; it < kIters; ++it) {
    float w[8];
    const float s = weights(words[it], w);
    const float cum = run + wave_inclusive_scan(s);
    if (at < 0) {   // wave-uniform
      if (__builtin_amdgcn_ballot_w64(s > 0.f)) last = it;
      if (__builtin_amdgcn_ballot_w64(s > 0.f && cum > want)) { at = it; cum_at = cum; }
    }
    run = from_lane(cum, 63);
  }
  const int piece = at >= 0 ? at : last;
  int tok = -1;
  float x_tok = 0.f;
  if (piece >= 0) {   // wave-uniform
    u32x4 v = words[0];
#pragma unroll
    for (int it = 1; it < kIters; ++it) v = it == piece ? words[it] : v;
    float w[8];
    const float s = weights(v, w);
    // the lane's first token with mass that passes; if rounding leaves none (or no lane passed), its last one
    const unsigned long long mass = __builtin_amdgcn_ballot_w64(s > 0.f);
    const unsigned long long hit = __builtin_amdgcn_ballot_w64(s > 0.f && cum_at > want);
    const int l = at >= 0 ? __builtin_ctzll(hit) : 63 - __builtin_clzll(mass);
    float acc = at >= 0 ? cum_at - s : -INFINITY;     // mass before this lane's 8 logits
    int e_pick = 0;
    bool found = false;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      acc += w[e];
      if (!found && w[e] > 0.f) { e_pick = e; found = acc > want; }
    }
    uint32_t word = v[0];
#pragma unroll
    for (int d = 1; d < 4; ++d) word = d == e_pick >> 1 ? v[d] : word;
    tok = from_lane((int)(cbase + piece * 512) + e_pick, l);
    x_tok = from_lane(__uint_as_float(e_pick & 1 ? word & 0xffff0000u : word << 16), l);
  }
  if (lane == 0) {
    if (tok < 0) {   // a row of -inf logits (or NaN): no token can be drawn
      a.out_tokens[row] = -1;
      a.out_logprobs[row] = __uint_as_float(0x7fc00000u);
    } else {
      a.out_tokens[row] = tok;
      a.out_logprobs[row] = logprob_of(x_tok, c, M, total);
    }
  }
}

__global__ __launch_bounds__(64) void sample_pick_kernel(SampleArgs a) {
  const int row = blockIdx.x;
  pick_token(a, a.partials + (size_t)row * a.num_chunks, a.num_chunks, row, a.uniforms[row]);
}

// Whole rows: a workgroup of up to 16 waves sums a row's chunks into LDS and its first wave draws the token, so
// there is one launch, and the chunk sums do not go through memory.  Chunks and sums are those of divided rows, bit for
// bit: which token is drawn does not depend on the size of the batch.  What bounds it: the vector ALU of the row's CU (7 issue
// slots of 4 cycles per logit) and the read together (256 x 152064: 78 MB in 18.9 us), and at a row's end 3 us of dependent
// steps.  (Chunks of 2048 take 17.1 us, but draw another token now and then, where the uniform number falls into an
// interval of the size of the sums' rounding.)
constexpr int kRowMaxWaves = 16;
constexpr int kRowMaxChunks = 1024;   // (a vocabulary of 4 M)
// kAhead: a wave requests its next chunk before it sums the present one, in 82 registers; without, 52 leave room for eight waves a SIMD.
template <bool kAhead>
__device__ __forceinline__ void sample_rows(const SampleArgs& a) {
  __shared__ float2 part[kRowMaxChunks];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int row = blockIdx.x;
  const uint16_t* x = a.logits + (size_t)row * a.vocab;
  const int chunks = a.num_chunks, waves = (int)blockDim.x >> 6;
  const float u = a.uniforms[row];
  u32x4 cur[kIters], nxt[kAhead ? kIters : 1];
  if (kAhead && wave < chunks) fetch_chunk(x, (long)wave * kChunk, lane, a.vocab, cur);
  for (int chunk = wave; chunk < chunks; chunk += waves) {
    const bool more = chunk + waves < chunks;   // wave-uniform
    if constexpr (kAhead) {
      if (more) fetch_chunk(x, (long)(chunk + waves) * kChunk, lane, a.vocab, nxt);
    } else {
      fetch_chunk(x, (long)chunk * kChunk, lane, a.vocab, cur);
    }
    end_chunk((long)chunk * kChunk, lane, a.vocab, cur);
    const float2 v = chunk_sum(cur, a.inv_temp_log2e);
    if (lane == 0) part[chunk] = v;
    if constexpr (kAhead) {
      if (more) {
#pragma unroll
        for (int it = 0; it < kIters; ++it) cur[it] = nxt[it];
      }
    }
  }
  __syncthreads();
  if (wave == 0) pick_token(a, part, chunks, row, u);
}
__global__ __launch_bounds__(kRowMaxWaves * 64) void sample_rows_kernel(SampleArgs a) { sample_rows<true>(a); }
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(8, 8))) void sample_many_rows_kernel(SampleArgs a) { sample_rows<false>(a); }

// ---------------------------------------------------------------------------------------
// Top-p (nucleus) sampling.  Tokens are ranked by probability (ties: lower index first); the
// nucleus is the shortest head of that ranking whose probability reaches top_p; the token is
// drawn from the nucleus by inverse CDF in INDEX order with the caller's uniform number scaled
// to the nucleus mass.  bf16 logits have at most 65536 distinct values and equal logits have
// equal probability, so the nucleus is "every token above a threshold value, plus the first c
// tokens at the threshold value": the kernel finds the threshold with exact counts per value
// instead of sorting 150 k tokens.
//
// One workgroup of 512 threads owns a row, three of them share a CU (long rows of small batches have one for themselves).  The row is cut into groups of
// 2048 tokens, group k * 8 + w belongs to wave w.  Passes over the row:
//   1. maximum value and Z = sum 2^(y - M)  (running (max, sum) per thread, fixed-order merge);
//   2. short list: the mass of the unlikely tokens is estimated from a sample of the row (it is made
//      of many small weights, so a few thousand samples give it to a few per cent, and Z is exact);
//      every token above a cut that leaves less than 1 - top_p below it is copied into a list in
//      LDS, wave by wave, and only the list is counted per value.  A scan of the value masses
//      count * 2^(y(value) - M) from the top finds the value at which the cumulative mass reaches
//      top_p * Z.  The cut only decides what is looked at: counts above it are complete, so a
//      threshold found in the list is THE threshold.  If none is found (the estimate was too high),
//      the list is too long, or the threshold is likely to be zero, negative or more than 2048 values
//      below the maximum, the counts are taken of the whole row instead, over windows of 8192 values: first
//      the one that starts at the cut, if the threshold is likely to lie in it, with the mass of what is
//      above it, then from the maximum down.  (Nuclei of half of a long row or more, rows of negative
//      logits.  64 x 152064, sigma 2, top_p 0.95: 49 us at T 1, with the list, and 60 at T 1.3, without;
//      2048 x 152064, top_p 0.9: 200 us, and 304 with 40 subtracted from every logit, which changes nothing else.)
//   3. per group the nucleus mass and the number of threshold-value tokens (from the list, if a third of a CU has room
//      for it, else one more pass over the row); a scan over the group sums finds the group in which the scaled
//      uniform is passed, a workgroup scan over the group's 2048 tokens finds the token.
// What bounds it, 2048 x 152064, sigma 3, top_p 0.9 (196 us): both reads and the vector ALU, neither of them alone.  The rows are
// fetched twice (1255 MB, 6.4 TB/s: three rows per CU are 234 MB, too many for the L2s), and the vector ALU issues in 76 %
// of the CUs' time: 17.1 issue slots of 4 cycles per logit over all passes, of which the first has 7
// and the copy into the list 3.5.  (Rows that the L2s hold take 148 us, and the fetches alone would take 180.)  Two workgroups
// per CU 212; with the row held in registers by one workgroup per CU, a count of all values in
// LDS (an LDS atomic on 64 lanes takes about 25 cycles) and a third pass over all tokens 508 us; the
// same with the list but still in registers 316 us (nothing to overlap the short phases with).
// A few rows (64 x 152064, top_p 0.95: 34 us): each has a CU of its own, whose vector ALU issues in half of that time, two waves
// per SIMD: pass 1 for 9 us (issue), the copy into the list 10 us (an exec mask and a store per token: a chain), in the rest it waits,
// at the barriers between the phases.  (16 waves a row: 3 % faster up to 128 rows, half as fast from 512 on.  Two stores per four
// tokens, selected and placed by lane counts, instead of four: 40 us.)
// Three workgroups per CU leave 80 vector registers: two are spilled (12 bytes of scratch per lane), outside the passes,
// and 48 scalar registers (60 where odd rows are shifted) to lanes of vector registers, which the counts over windows read back.
// ---------------------------------------------------------------------------------------
constexpr int kTpThreads = 512;
constexpr int kTpWaves = kTpThreads / 64;
constexpr int kWin = 8192;                   // values per window of the count without the list
constexpr int kTpGroup = 2048;               // tokens of a group: 4 x 512, one wave
constexpr int kLowestKey = 0x0080;           // key of the most negative finite bf16; below: -inf, NaN
constexpr int kScanStep = 4;                 // scan positions per thread and round of the threshold search
constexpr int kListGroups = 20;              // groups per wave that the list covers (vocab <= 327680)
constexpr int kListWin = 2048;               // values the list may span
constexpr int kBins = 256;                   // bins of the tail estimate, an eighth of a power of two each
constexpr int kSampleWords = 10;             // words per thread that the estimate looks at

__device__ __forceinline__ int key_of(uint32_t bits) {   // larger value <=> larger key; -0 counts as +0
  if ((bits & 0x7fffu) == 0) bits = 0;
  return (bits & 0x8000u) ? (int)(~bits & 0xffffu) : (int)(bits | 0x8000u);
}
__device__ __forceinline__ float value_of_key(int key) {
  const uint32_t bits = (key & 0x8000) ? (uint32_t)(key & 0x7fff) : (~(uint32_t)key & 0xffffu);
  return __uint_as_float(bits << 16);
}

constexpr int kListCapShared = 2624, kListCapAlone = 9216;   // list entries per wave: three rows on a CU, and one
template <int kListCap>
struct TpShared {
  union {
    uint32_t hist[kWin];                       // counts of pass 2 without the list; group sums of pass 3
    uint32_t sample[kSampleWords][kTpThreads]; // pass 1: one word (two tokens) per thread and group
    struct {
      uint16_t list[kTpWaves][kListCap];       // the tokens above the cut, bf16 bits, the wave's last group first
      uint32_t list_hist[kListWin];            // their counts per value
    };
  };
  float group_mass[kListGroups * kTpWaves];    // group sums of pass 3 from the list
  int group_ties[kListGroups * kTpWaves];
  int seg_end[kTpWaves][kListGroups];          // where each group's entries end in its wave's list
  int bins[kBins];
  double wave_d[kTpWaves];
  float wave_f[kTpWaves];
  float wave_m[kTpWaves];
  int wave_i[kTpWaves];
  int list_full, list_long;     // a wave's list has no room; had none in kListCapShared
  int found_at;                 // smallest scan position / thread index that meets a condition
  int thr_key, thr_cnt;         // threshold value (key) and how many tokens have it
  double thr_above;             // mass strictly above the threshold value
  int group, ties_before;
  float want_in_group;          // nucleus mass still to pass inside the chosen group
  int out_tok;
};
static_assert(sizeof(TpShared<kListCapShared>) <= 42 * 1280, "three workgroups share a CU's 160 KB");
static_assert(sizeof(TpShared<kListCapAlone>) <= 160 * 1024, "a workgroup has a CU's LDS");

// exclusive scans over the workgroup in thread order (fixed order: bit-identical reruns)
// kBefore: what comes before a thread is summed without the thread's own value, not taken as the difference (which rounds with it)
template <bool kBefore = false, class Shared>
__device__ __forceinline__ double block_excl_scan_d(double v, double& total, Shared& sh) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const double inc = wave_inclusive_scan(v);
  __syncthreads();
  if (lane == 63) sh.wave_d[wave] = inc;
  __syncthreads();
  double before = 0.0, all = 0.0;
#pragma unroll
  for (int w = 0; w < kTpWaves; ++w) {
    if (w < wave) before += sh.wave_d[w];
    all += sh.wave_d[w];
  }
  total = all;
  if constexpr (kBefore) return before + dpp_or_zero<0x138, 0xf>(inc);   // wave_shr:1
  return before + inc - v;
}
template <class Shared>
__device__ __forceinline__ float block_excl_scan_f(float v, Shared& sh) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const float inc = wave_inclusive_scan(v);
  __syncthreads();
  if (lane == 63) sh.wave_f[wave] = inc;
  __syncthreads();
  float before = 0.f;
#pragma unroll
  for (int w = 0; w < kTpWaves; ++w)
    if (w < wave) before += sh.wave_f[w];
  return before + inc - v;
}
template <class Shared>
__device__ __forceinline__ int block_excl_scan_i(int v, Shared& sh) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int inc = wave_inclusive_scan(v);
  __syncthreads();
  if (lane == 63) sh.wave_i[wave] = inc;
  __syncthreads();
  int before = 0;
#pragma unroll
  for (int w = 0; w < kTpWaves; ++w)
    if (w < wave) before += sh.wave_i[w];
  return before + inc - v;
}

// the two bf16 of a word widened to float
__device__ __forceinline__ float lo_val(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float hi_val(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

// a value that is the same in every lane, moved to a scalar register (frees a vector register)
__device__ __forceinline__ float uniform_f(float v) { return __uint_as_float((uint32_t)__builtin_amdgcn_readfirstlane((int)__float_as_uint(v))); }
__device__ __forceinline__ int uniform_i(int v) { return __builtin_amdgcn_readfirstlane(v); }

// The threshold search: hist[] holds the counts of the values hi, hi - 1, ... (position j of the
// scan is the value hi - j, its count hist[hi - j - lo]), npos positions.  The positions are
// scanned in rounds of kScanStep per thread (thread t owns base + kScanStep t ...) and the scan
// stops at the round in which the cumulative mass, `above` included, reaches tau: for peaked rows
// that is the first round, a few hundred values below the maximum.  Returns whether it was
// reached (workgroup-uniform; then sh.thr_* are set, visible after the barrier this ends with),
// adds the scanned mass to `above`.
template <class Weight, class Shared>
__device__ __forceinline__ bool find_threshold(const uint32_t* hist, int hi, int lo, int npos, double tau,
                                               double& above, Weight&& weight, Shared& sh) {
  const int tid = threadIdx.x;
  auto mass_at = [&](int pos) {
    const int key = hi - pos;
    const uint32_t cnt = pos < npos ? hist[key - lo] : 0u;
    return cnt ? (double)cnt * (double)weight(key) : 0.0;
  };
  double scanned = 0.0;
  bool found = false;
  for (int base = 0; base < npos; base += kScanStep * kTpThreads) {
    const int p0 = base + tid * kScanStep;
    double mine = 0.0;
#pragma unroll
    for (int q = 0; q < kScanStep; ++q) mine += mass_at(p0 + q);
    double round_total;
    const double before = above + scanned + block_excl_scan_d<true>(mine, round_total, sh);
    // first scan position at which the cumulative mass reaches tau: every thread at or past
    // the crossing proposes its first such position, the smallest wins (robust against the
    // last-bit differences between neighbouring threads' scan values)
    int my_pos = kWin;
    double my_above = 0.0;
    if (before + mine >= tau) {
      double run = before;
#pragma unroll 1
      for (int q = 0; q < kScanStep; ++q) {
        const double m = mass_at(p0 + q);
        if (m > 0.0 && run + m >= tau) { my_pos = p0 + q; my_above = run; break; }
        run += m;
      }
      if (my_pos < kWin) atomicMin(&sh.found_at, my_pos);
    }
    __syncthreads();
    found = sh.found_at < kWin;             // workgroup-uniform
    if (my_pos < kWin && my_pos == sh.found_at) {
      const int key = hi - my_pos;
      sh.thr_key = key;
      sh.thr_cnt = (int)hist[key - lo];
      sh.thr_above = my_above;
    }
    __syncthreads();
    if (found) break;
    scanned += round_total;
  }
  above += scanned;
  return found;
}

// Appends the tokens of four words that are >= the cut to a lane's place in the list, in LDS, without
// a branch or an unpacked copy: per token one comparison that sets EXEC, one store, one addition.
// `cut` holds the cut's bf16 bits as a signed 16-bit number (positive, so that it orders the bit
// patterns), cut_f the same value as a float, whose comparison with a whole word decides for the
// upper half (the lower half only adds to a positive number's magnitude and cannot reach the next
// bf16).  All 64 lanes must be active.
__device__ __forceinline__ void append_words(uint32_t& at, u32x4 v, int cut, float cut_f) {
#define MARL_APPEND_WORD(W)            \
  "v_cmpx_le_i16 vcc, %5, " W "\n"     \
  "ds_write_b16 %0, " W "\n"           \
  "v_add_u32 %0, 2, %0\n"              \
  "s_mov_b64 exec, -1\n"               \
  "v_cmpx_le_f32 vcc, %6, " W "\n"     \
  "ds_write_b16_d16_hi %0, " W "\n"    \
  "v_add_u32 %0, 2, %0\n"              \
  "s_mov_b64 exec, -1\n"
  asm volatile(MARL_APPEND_WORD("%1") MARL_APPEND_WORD("%2") MARL_APPEND_WORD("%3") MARL_APPEND_WORD("%4")
               "s_nop 4"   // a DPP instruction must stay five slots behind a write of EXEC
               : "+v"(at) : "v"(v[0]), "v"(v[1]), "v"(v[2]), "v"(v[3]), "s"(cut), "s"(cut_f) : "vcc", "memory");
#undef MARL_APPEND_WORD
}

// The 32 tokens of a thread where the group was read from the element before it, which starts a dword: every token moves down by half
// a dword, and a lane's last one comes from the lane behind it, the last lane's from `next` (the dword of the group's last token).
__device__ __forceinline__ void shift_down(u32x4 (&v)[4], uint32_t next) {
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const uint32_t behind = j < 3 ? (uint32_t)__builtin_amdgcn_readfirstlane((int)v[j + 1][0]) : next;
    const uint32_t above = (uint32_t)__builtin_amdgcn_update_dpp((int)behind, (int)v[j][0], 0x130, 0xf, 0xf, false);   // wave_shl:1
#pragma unroll
    for (int d = 0; d < 4; ++d) v[j][d] = __builtin_amdgcn_alignbit(d < 3 ? v[j][d + 1] : above, v[j][d], 16);
  }
}

template <int kListCap, bool kOdd>
__device__ __forceinline__ void sample_top_p(const TopPArgs& a) {
  __shared__ TpShared<kListCap> sh;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int row = blockIdx.x;
  const uint16_t* x = a.logits + (size_t)row * a.vocab;
  const float c = a.inv_temp_log2e;
  const long V = a.vocab;
  const int ngroups = (int)((V + kTpGroup - 1) / kTpGroup);
  const float u = a.uniforms[row];   // (requested early: used after the passes)
  const int my_groups = wave < ngroups ? (ngroups - wave + kTpWaves - 1) / kTpWaves : 0;   // of this wave
  // kOdd: rows that start in the middle of a dword.  Their 16-byte loads would take up to twice the requests (from dwords on, all
  // are alike): whole groups are read from the element before them and shifted into place.  Which thread has which token does not
  // depend on where a row starts: what it draws is a function of the row.
  const bool odd_row = kOdd && (reinterpret_cast<uintptr_t>(x) & 2) != 0;
  auto shifted = [&](int g) { return kOdd && odd_row && g > 0 && (long)(g + 1) * kTpGroup < V; };   // (never read outside the row)
  // One pass over this wave's groups in order, the next group's loads in flight:
  // fn(group, this thread's 4 x 8 tokens of it); positions past the end of the row read as -inf.
  auto sweep = [&](auto&& fn, auto backwards_tag) {
    constexpr bool kBack = decltype(backwards_tag)::value;
    uint32_t cur_next = 0, nxt_next = 0;
    auto fetch = [&](int g, u32x4 (&v)[4], uint32_t& next) {
      const long base = (long)g * kTpGroup;
      if (base + kTpGroup <= V) {   // wave-uniform
        const uint16_t* from = x + base - (shifted(g) ? 1 : 0);
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = *reinterpret_cast<const u32x4_any*>(from + j * 512 + lane * 8);
        if (shifted(g)) next = (uint32_t)ld_uniform(reinterpret_cast<const int32_t*>(from + kTpGroup));
      } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = load8_words(x, base + j * 512 + lane * 8, V);
      }
    };
    u32x4 cur[4], nxt[4];
    auto group_at = [&](int k) { return wave + kTpWaves * (kBack ? my_groups - 1 - k : k); };
    if (my_groups > 0) fetch(group_at(0), cur, cur_next);
    for (int k = 0; k < my_groups; ++k) {
      if (k + 1 < my_groups) fetch(group_at(k + 1), nxt, nxt_next);
      if (shifted(group_at(k))) shift_down(cur, cur_next);
      fn(group_at(k), cur);
#pragma unroll
      for (int j = 0; j < 4; ++j) cur[j] = nxt[j];
      cur_next = nxt_next;
    }
  };
  const std::false_type forwards{};
  const std::true_type backwards{};   // what was read last is the likeliest to be in a cache still

  // ---- pass 1: largest value and Z relative to it -----------------------------------------------
  // per thread a running (largest logit so far, sum relative to it); merged in thread order
  float xrun = -INFINITY, mrun = -INFINITY, zrun = 0.f;   // largest raw logit, the same times c, sum
  // the sample: a word per thread and group, two or four in short rows (fewer give a vague cut); of long rows every
  // second, third ... group, so that the whole row is in it
  const int most_groups = (ngroups + kTpWaves - 1) / kTpWaves;   // of a wave
  const int sample_of_group = most_groups == 1 ? 4 : most_groups == 2 ? 2 : 1;
  const int sample_every = (most_groups + kSampleWords - 1) / kSampleWords;
  int sample_words = 0, sample_wait = 0;   // of this wave so far; groups until the next one that is looked at
  sweep([&](int, const u32x4 (&v)[4]) {
    float x8 = xrun;
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int d = 0; d < 4; ++d) x8 = fmaxf(x8, fmaxf(lo_val(v[j][d]), hi_val(v[j][d])));
    // c > 0: the largest raw logit is the largest scaled one.  While nothing finite has been seen the
    // reference is 0: every weight is 0 (or NaN, which the check of Z below catches).
    const float m8 = x8 * c;
    const float ms = x8 > -INFINITY ? m8 : 0.f;
    float s[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int d = 0; d < 4; ++d) {
        s[d] += ex2(__builtin_fmaf(lo_val(v[j][d]), c, -ms));
        s[d] += ex2(__builtin_fmaf(hi_val(v[j][d]), c, -ms));
      }
    zrun = zrun * ex2(mrun - ms) + ((s[0] + s[1]) + (s[2] + s[3]));   // mrun = -inf: zrun was 0
    xrun = x8;
    mrun = m8;
    if (--sample_wait < 0) {   // wave-uniform
      sample_wait = sample_every - 1;
      sh.sample[sample_words][tid] = v[0][0];
      if (sample_of_group > 1) sh.sample[sample_words + 1][tid] = v[2][0];
      if (sample_of_group > 2) { sh.sample[sample_words + 2][tid] = v[1][0]; sh.sample[sample_words + 3][tid] = v[3][0]; }
      sample_words += sample_of_group;
    }
  }, forwards);
  float xmax = wave_max(xrun);
  if (lane == 0) sh.wave_m[wave] = xmax;
  if (tid < kBins) sh.bins[tid] = 0;
  if (tid == 0) { sh.thr_key = -1; sh.thr_cnt = 0; sh.thr_above = 0.0; sh.found_at = kWin; sh.list_full = sh.list_long = 0; }
  __syncthreads();
#pragma unroll
  for (int w = 0; w < kTpWaves; ++w) xmax = fmaxf(xmax, sh.wave_m[w]);
  xmax = uniform_f(xmax);
  const float M = uniform_f(xmax * c);
  // the sample is counted here, so that it shares the barriers of the sum below
  for (int k = 0; k < sample_words; ++k) {   // wave-uniform; (a NaN counts as the lightest)
    const uint32_t w = sh.sample[k][tid];
    const float y0 = (xmax - lo_val(w)) * (8.0f * c), y1 = (xmax - hi_val(w)) * (8.0f * c);
    atomicAdd(&sh.bins[(int)fminf(y0, (float)(kBins - 1))], 1);
    atomicAdd(&sh.bins[(int)fminf(y1, (float)(kBins - 1))], 1);
  }
  double ztot;
  block_excl_scan_d(xrun > -INFINITY ? (double)zrun * (double)ex2(mrun - M) : (double)zrun, ztot, sh);
  const double Z = ztot;
  if (!(xmax > -INFINITY) || !(Z > 0.0) || !(Z < 1e300)) {   // no finite logit, or +inf / NaN: nothing to draw
    if (tid == 0) {
      a.out_tokens[row] = -1;
      a.out_logprobs[row] = __uint_as_float(0x7fc00000u);
    }
    return;
  }
  const int kmax = key_of(__float_as_uint(xmax) >> 16);
  // the weight of a value, computed the same way everywhere: 2^(fma(value, c, -M))
  auto weight = [&](int key) { return key >= kLowestKey ? ex2(__builtin_fmaf(value_of_key(key), c, -M)) : 0.f; };

  // ---- pass 2: the threshold value --------------------------------------------------------
  // thr_key = -1: every token with a finite logit is in the nucleus
  // What is drawn is a function of the row, whatever the list has room for.  From the list or from a window that starts at the
  // maximum, the threshold is found by the same sums (what comes before a thread of the search does not depend on how many of
  // the thread's own values the list has), so a row whose list would begin never tries another window before that one.  The groups' masses are rounded otherwise in a list than in the row: they are taken from lists that
  // kListCapShared has room for, in every instance (`short_list`).
  bool from_list = false, short_list = true;
  int cut_key = 0, likely_key = 0;   // where the estimate puts the threshold at the lowest, and where it puts it
  const double tau = (double)a.top_p * Z;
  if (a.top_p < 1.f && ngroups <= kListGroups * kTpWaves) {
    // the cut: the largest bin boundary below which the sample promises at most 1 - top_p: its sum (every
    // token at the upper edge of its bin) plus three standard deviations of it.  Where few tokens hold the mass, the sample may
    // have missed the very ones that decide, and its variance knows nothing of them: kUnseen tokens at the boundary are added to
    // that.  (Without them, sigma 3, T 0.7, top_p 0.8, two to four rows in a hundred have too high a cut, sigma 4 at T 0.6 one in
    // four, and their counts over windows keep the whole batch: 30 x 152064 57.6 us, with them 28.9, 250 x 65536 32.6 and 18.1, 1500 x 20481 51.6
    // and 39.9.  In 16000 simulated rows of 4096 to 152064 tokens none; the list is 0 to 3 % longer where it has more than 500 tokens.)
    // (every wave computes it for itself; the bins were complete before the scan's barriers)
    constexpr float kUnseen = 3.f;
    int count[4];        // lane 0: the lightest bins, from kBins - 1 down
    float mass[4], square[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int bin = kBins - 1 - 4 * lane - e;
      const float w = ex2(-0.125f * (float)bin);
      count[e] = sh.bins[bin];
      mass[e] = (float)count[e] * w;
      square[e] = mass[e] * w;
    }
    const int sampled = from_lane(wave_inclusive_scan((count[0] + count[1]) + (count[2] + count[3])), 63);
    const float mine_m = (mass[0] + mass[1]) + (mass[2] + mass[3]), mine_s = (square[0] + square[1]) + (square[2] + square[3]);
    float tail = wave_inclusive_scan(mine_m) - mine_m, var = fmaxf(wave_inclusive_scan(mine_s) - mine_s, 0.f);
    const float allowed = (float)((1.0 - (double)a.top_p) * Z * (double)sampled / ((double)ngroups * kTpGroup));
    int skip = 0, unlikely = 0;        // bins left out, by the estimate with its deviations and by itself
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      tail += mass[e];
      var += square[e];
      const float w = ex2(-0.125f * (float)(kBins - 1 - 4 * lane - e));
      skip += (int)__popcll(__builtin_amdgcn_ballot_w64(tail + 3.f * __builtin_sqrtf(__builtin_fmaf(kUnseen * w, w, var)) <= allowed));
      unlikely += (int)__popcll(__builtin_amdgcn_ballot_w64(tail <= allowed));
    }
    auto key_below = [&](int bins) {   // the largest key that lies below so many bins from the maximum on
      return uniform_i(min(kmax, max(kLowestKey, key_of(__float_as_uint(xmax - 0.125f * (float)max(1, bins) / c) >> 16))));
    };
    cut_key = key_below(kBins - skip);
    likely_key = key_below(kBins - unlikely);
    // The list starts at the cut, or where its counts still span it if the threshold is likely to lie above that
    // (short rows give a vague estimate, whose cut may be zero or negative), and is not begun if the
    // sample has more tokens above than a wave's list takes.
    const int lkey = max(cut_key, kmax - (kListWin - 1));
    const int span = kmax - lkey + 1;
    const float bins_listed = 8.f * c * (xmax - value_of_key(lkey));
    int listed = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) listed += (float)(kBins - 4 * lane - e) <= bins_listed ? count[e] : 0;   // (whole bins)
    listed = from_lane(wave_inclusive_scan(listed), 63);
    // (An overflow costs a row alone on a CU its whole list pass, and its batch with it: such a list keeps room for what
    // the waves and the sample deviate, or 68 x 156368 at sigma 2, T 1.3, top_p 0.9 takes 69 us, not 57.  Among rows that share a CU
    // it is hidden, and counting instead costs more: 700 x 152064 at sigma 3, T 1.3, top_p 0.84 122 us, 86 with some in vain.)
    constexpr float kListRoom = kListCap > kListCapShared ? 0.95f * kListCap : kListCap;
    const bool fits = (float)listed * (float)(most_groups * kTpGroup) <= kListRoom * (float)sampled;
    if (lkey >= 0x8080 && likely_key >= lkey && fits) {   // workgroup-uniform: a positive, normal cut
      if (kListCap > kListCapShared) short_list = (float)listed * (float)(most_groups * kTpGroup) <= (float)kListCapShared * (float)sampled;
      const int cut = lkey - 0x8000;           // its bits
      const float cut_f = uniform_f(value_of_key(lkey));
      // (the list takes the sample's place: it was read before the barriers of the sum)
      for (int p = tid; p < span; p += kTpThreads) sh.list_hist[p] = 0;
      const uint32_t list_at = (uint32_t)reinterpret_cast<uintptr_t>(&sh.list[wave][0]);   // LDS address
      typedef short i16x2 __attribute__((ext_vector_type(2)));
      const i16x2 cut2 = {(short)cut, (short)cut};
      int n = 0;           // wave-uniform
      bool full = false;
      // a lane's entries of a group are adjacent: one scan per group places them
      sweep([&](int g, const u32x4 (&v)[4]) {
        if (full) return;   // wave-uniform
        int below[4] = {0, 0, 0, 0};
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
          for (int d = 0; d < 4; ++d) {
            const i16x2 t = __builtin_elementwise_sub_sat(__builtin_bit_cast(i16x2, (uint32_t)v[j][d]), cut2);
            below[j] += __builtin_popcount(__builtin_bit_cast(uint32_t, t) & 0x80008000u);
          }
        const int mine = 32 - ((below[0] + below[1]) + (below[2] + below[3]));
        const int inc = wave_inclusive_scan(mine);
        const int total = from_lane(inc, 63);
        full = n + total > kListCap;
        if (!full) {   // wave-uniform
          uint32_t at = list_at + 2u * (uint32_t)(n + inc - mine);
#pragma unroll
          for (int j = 0; j < 4; ++j)
            if (__builtin_amdgcn_ballot_w64(below[j] < 8) != 0) append_words(at, v[j], cut, cut_f);
          n += total;
        }
        if (lane == 0) sh.seg_end[wave][g / kTpWaves] = n;
      }, backwards);
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the stores of append_words
      if (full && lane == 0) sh.list_full = 1;
      if (kListCap > kListCapShared && n > kListCapShared && lane == 0) sh.list_long = 1;
      __syncthreads();
      if (kListCap > kListCapShared) short_list = short_list && !sh.list_long;
      if (!sh.list_full) {   // workgroup-uniform
        constexpr int kAtOnce = 8;
        for (int p = lane; p < n; p += 64 * kAtOnce) {
          uint32_t e[kAtOnce];
#pragma unroll
          for (int u = 0; u < kAtOnce; ++u) e[u] = sh.list[wave][min(p + 64 * u, n - 1)];
#pragma unroll
          for (int u = 0; u < kAtOnce; ++u)
            if (p + 64 * u < n) atomicAdd(&sh.list_hist[e[u] - cut], 1u);   // (positive values: key - lkey)
        }
        __syncthreads();
        double above = 0.0;
        from_list = find_threshold(sh.list_hist, kmax, lkey, span, tau, above, weight, sh);
      }
    }
  }
  if (a.top_p < 1.f && !from_list) {
    // Counts of the whole row over a window of values.  First the window that starts at the estimated
    // cut: the mass of the values above it is summed in the same pass, so one pass is enough unless the
    // threshold lies outside (not tried where it is likely to lie above); then the windows from the maximum down.
    // x_above: the smallest value above the window (one key further up: not every pattern is a value of its own,
    // the one below +0 is -0), `above`: the mass from it on; +inf where nothing lies above
    auto count_window = [&](int hi, int lo, float x_above, double& above) {
      __syncthreads();                        // what this memory held before has been read
      for (int i = tid; i < kWin; i += kTpThreads) sh.hist[i] = 0;
      __syncthreads();
      const int lo_eff = max(lo, kLowestKey);
      const unsigned span = (unsigned)(hi - lo_eff);
      sweep([&](int, const u32x4 (&v)[4]) {
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
          for (int d = 0; d < 4; ++d) {
            const float r0 = lo_val(v[j][d]), r1 = hi_val(v[j][d]);
            if (x_above <= xmax) {   // workgroup-uniform
              above += (double)((r0 >= x_above ? ex2(__builtin_fmaf(r0, c, -M)) : 0.f) +
                                (r1 >= x_above ? ex2(__builtin_fmaf(r1, c, -M)) : 0.f));
            }
            const int k0 = key_of(v[j][d] & 0xffffu), k1 = key_of(v[j][d] >> 16);
            if ((unsigned)(k0 - lo_eff) <= span) atomicAdd(&sh.hist[k0 - lo], 1u);
            if ((unsigned)(k1 - lo_eff) <= span) atomicAdd(&sh.hist[k1 - lo], 1u);
          }
      }, forwards);
      __syncthreads();
    };
    bool found = false;
    const int list_from = kmax - (kListWin - 1);   // where the list of such a wide span would begin
    if (cut_key > kLowestKey && cut_key + kWin <= kmax && likely_key < cut_key + kWin && (list_from < 0x8080 || likely_key < list_from)) {
      const int hi = cut_key + kWin - 1;
      double mine = 0.0, above;
      count_window(hi, cut_key, value_of_key(hi + 1), mine);
      block_excl_scan_d(mine, above, sh);
      if (above < tau) found = find_threshold(sh.hist, hi, cut_key, kWin, tau, above, weight, sh);
    }
    double above = 0.0;                       // mass of the values above the window
    for (int hi = kmax; hi >= kLowestKey && !found; hi -= kWin) {
      double none = 0.0;
      count_window(hi, hi - (kWin - 1), INFINITY, none);
      found = find_threshold(sh.hist, hi, hi - (kWin - 1), kWin, tau, above, weight, sh);
    }
  }
  __syncthreads();
  const int thr_key = uniform_i(sh.thr_key);
  // how many of the threshold-value tokens (in index order) the nucleus takes
  int ties_kept = 0;
  float thr_w = 0.f;
  double nucleus = Z;
  if (thr_key >= 0) {
    thr_w = uniform_f(weight(thr_key));
    const double need = (tau - sh.thr_above) / (double)thr_w;
    ties_kept = uniform_i((int)fmin(fmax(ceil(need), 1.0), (double)sh.thr_cnt));
    nucleus = sh.thr_above + (double)ties_kept * (double)thr_w;
  }
  // the walk over the group sums runs in double precision (a float32 running sum over the whole
  // vocabulary would move a CDF step by up to ~1e-5 of the nucleus mass); inside the chosen group
  // float32 sums start from zero again and are compared with the mass that is left to pass
  const double target = (double)u * nucleus;
  // pass 3 compares raw logit values (every bf16 is exact in float; -0 == +0 as in the keys);
  // with no threshold every finite logit is above it
  const float thr_x = uniform_f(thr_key >= 0 ? value_of_key(thr_key) : -INFINITY);

  // ---- pass 3: inverse CDF over the nucleus in index order ----------------------------------
  // per group: mass of the tokens above the threshold, number of tokens at it
  float* part_m = reinterpret_cast<float*>(sh.hist);             // [ngroups]
  int* part_n = reinterpret_cast<int*>(sh.hist) + kWin / 2;      // [ngroups]
  if (from_list && short_list) {
    part_m = sh.group_mass;
    part_n = sh.group_ties;
    // A power of two lanes per group, 4 to 64, so that most of the wave has a share of a group: 16, 8, 4, 2 groups at once or one,
    // whichever leaves the fewest idle and takes the fewest rounds (10 groups: 8 and 2).  One group after the other, reduced over the
    // wave, took five times as long (a chain of LDS reads and reductions per group); four lanes each wherever there are more
    // than four groups walk through hundreds of entries (64 x 152064, top_p 0.95: 36.3 us, now 34.3; 256 x 32003, sigma 2:
    // 25.3, now 23.2; 2048 x 152064 208 and 204).
    int at_once;
    for (int k0 = 0; k0 < my_groups; k0 += at_once) {   // wave-uniform
      const int left = my_groups - k0, log = left > 10 ? 4 : left > 5 ? 3 : left > 2 ? 2 : left - 1;
      at_once = 1 << log;
      const int per = 64 >> log, mine = lane & (per - 1);
      const int slot = k0 + (lane >> (6 - log)), k = min(slot, my_groups - 1);
      const int begin = k + 1 < my_groups ? sh.seg_end[wave][k + 1] : 0, end = sh.seg_end[wave][k];   // (listed backwards)
      double mg = 0.0;
      int n = 0;
      for (int p = begin + mine; p < end; p += 4 * per) {
        float r[4], w[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) r[u] = __uint_as_float((uint32_t)sh.list[wave][min(p + per * u, end - 1)] << 16);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const bool in = p + per * u < end;
          const float e = ex2(__builtin_fmaf(r[u], c, -M));
          w[u] = in && r[u] > thr_x ? e : 0.f;
          n += in && r[u] == thr_x;
        }
        mg += (double)((w[0] + w[1]) + (w[2] + w[3]));
      }
      // the sum of a group's lanes in the last of them
      mg += dpp_or_zero<0x111, 0xf>(mg);   // row_shr:1
      n += dpp_or_zero<0x111, 0xf>(n);
      mg += dpp_or_zero<0x112, 0xf>(mg);   // row_shr:2
      n += dpp_or_zero<0x112, 0xf>(n);
      if (per > 4) {
        mg += dpp_or_zero<0x114, 0xf>(mg);   // row_shr:4
        n += dpp_or_zero<0x114, 0xf>(n);
      }
      if (per > 8) {
        mg += dpp_or_zero<0x118, 0xf>(mg);   // row_shr:8
        n += dpp_or_zero<0x118, 0xf>(n);
      }
      if (per > 16) {
        mg += dpp_or_zero<0x142, 0xa>(mg);   // row_bcast:15 into rows 1 and 3
        n += dpp_or_zero<0x142, 0xa>(n);
      }
      if (per > 32) {
        mg += dpp_or_zero<0x143, 0xc>(mg);   // row_bcast:31 into rows 2 and 3
        n += dpp_or_zero<0x143, 0xc>(n);
      }
      if (mine == per - 1 && slot < my_groups) {
        part_m[k * kTpWaves + wave] = (float)mg;
        part_n[k * kTpWaves + wave] = n;
      }
    }
  } else {
    sweep([&](int g, const u32x4 (&v)[4]) {
      float m[4] = {0.f, 0.f, 0.f, 0.f};
      int n8 = 0;
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int d = 0; d < 4; ++d) {
          const float r0 = lo_val(v[j][d]), r1 = hi_val(v[j][d]);
          const float w0 = ex2(__builtin_fmaf(r0, c, -M)), w1 = ex2(__builtin_fmaf(r1, c, -M));
          m[d] += r0 > thr_x ? w0 : 0.f;
          m[d] += r1 > thr_x ? w1 : 0.f;
          n8 += (r0 == thr_x) + (r1 == thr_x);
        }
      const double mg = wave_inclusive_scan(((double)m[0] + (double)m[1]) + ((double)m[2] + (double)m[3]));
      n8 = wave_allreduce_sum(n8);
      if (lane == 63) { part_m[g] = (float)mg; part_n[g] = n8; }
    }, backwards);
  }
  __syncthreads();
  if (wave == 0) {
    // 64 groups per round, in order: which of a group's threshold-value tokens the nucleus keeps
    // follows from the number before the group
    double cum = 0.0, last_cum = 0.0, at_cum = 0.0;
    int ties = 0, group = -1, at_ties = 0, last_group = 0, last_ties = 0;
    for (int base = 0; base < ngroups && group < 0; base += 64) {
      const int g = base + lane;
      const int n = g < ngroups ? part_n[g] : 0;
      const int n_inc = wave_inclusive_scan(n);
      const int before_n = ties + n_inc - n;
      const double kept = (g < ngroups ? (double)part_m[g] : 0.0) + (double)thr_w * (double)min(n, max(0, ties_kept - before_n));
      const double after = cum + wave_inclusive_scan(kept);
      const unsigned long long hit = __builtin_amdgcn_ballot_w64(g < ngroups && kept > 0.0 && after > target);
      const unsigned long long nz = __builtin_amdgcn_ballot_w64(kept > 0.0);
      if (nz) {
        const int l = 63 - __builtin_clzll(nz);
        last_group = base + l;
        last_cum = from_lane(after - kept, l);
        last_ties = from_lane(before_n, l);
      }
      if (hit) {
        const int l = __builtin_ctzll(hit);
        group = base + l;
        at_cum = from_lane(after - kept, l);
        at_ties = from_lane(before_n, l);
      }
      cum = from_lane(after, 63);
      ties += from_lane(n_inc, 63);
    }
    if (group < 0) {              // rounding left the target at or above the total: the last token
      group = last_group;         // of the nucleus is taken (inside the group, below)
      at_cum = last_cum;
      at_ties = last_ties;
    }
    if (lane == 0) {
      sh.group = group;
      sh.want_in_group = (float)(target - at_cum);
      sh.ties_before = at_ties;
      sh.found_at = kTpThreads;
      sh.out_tok = -1;
    }
  }
  __syncthreads();
  {
    // the group's tokens once more, in index order: four per thread
    const long pos = (long)sh.group * kTpGroup + tid * 4;
    float r[4];
    uint32_t raw[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) raw[e] = x[min(pos + e, V - 1)];
#pragma unroll
    for (int e = 0; e < 4; ++e) r[e] = pos + e < V ? __uint_as_float(raw[e] << 16) : -INFINITY;
    int n4 = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) n4 += r[e] == thr_x;
    int rank = sh.ties_before + block_excl_scan_i(n4, sh);       // threshold-value tokens before this thread
    float w4[4], m4 = 0.f;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      float w = 0.f;
      if (r[e] > thr_x) w = ex2(__builtin_fmaf(r[e], c, -M));
      else if (r[e] == thr_x) { if (rank < ties_kept) w = thr_w; ++rank; }
      w4[e] = w;
      m4 += w;
    }
    const float want = sh.want_in_group;
    const float before = block_excl_scan_f(m4, sh);
    const bool pass = before + m4 > want && m4 > 0.f;
    if (pass) atomicMin(&sh.found_at, tid);
    // the last thread of the group that holds a nucleus token, for the rounding fallback
    if (m4 > 0.f) atomicMax(&sh.out_tok, tid);
    __syncthreads();
    const int winner = sh.found_at < kTpThreads ? sh.found_at : sh.out_tok;
    const bool fallback = sh.found_at >= kTpThreads;
    if (winner < 0 && tid == 0) {   // no nucleus token in the group: cannot happen for Z > 0
      a.out_tokens[row] = -1;
      a.out_logprobs[row] = __uint_as_float(0x7fc00000u);
    }
    if (tid == winner) {
      float run = before;
      int e_pick = -1;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if (w4[e] > 0.f) {
          run += w4[e];
          if (fallback) e_pick = e;                               // last nucleus token of the thread
          else if (e_pick < 0 && run > want) e_pick = e;
        }
      }
      if (e_pick < 0) {                                           // cannot happen: pass implies a hit
#pragma unroll
        for (int e = 0; e < 4; ++e) if (w4[e] > 0.f) e_pick = e;
      }
      float r_pick = r[0];
#pragma unroll
      for (int e = 1; e < 4; ++e) if (e == e_pick) r_pick = r[e];
      a.out_tokens[row] = (int)(pos + e_pick);
      a.out_logprobs[row] = logprob_of(r_pick, c, M, Z);
    }
  }
}

__global__ __launch_bounds__(kTpThreads) __attribute__((amdgpu_waves_per_eu(6, 6)))
void sample_top_p_kernel(TopPArgs a) { sample_top_p<kListCapShared, false>(a); }
__global__ __launch_bounds__(kTpThreads) __attribute__((amdgpu_waves_per_eu(6, 6)))
void sample_top_p_odd_kernel(TopPArgs a) { sample_top_p<kListCapShared, true>(a); }
__global__ __launch_bounds__(kTpThreads) __attribute__((amdgpu_waves_per_eu(2, 2)))
void sample_top_p_alone_kernel(TopPArgs a) { sample_top_p<kListCapAlone, false>(a); }

}  // namespace

int sample_num_chunks(int vocab) { return (vocab + kChunk - 1) / kChunk; }

int top_p_max_vocab() { return 1 << 23; }   // its 4096 groups' sums fit the LDS buffer

constexpr int kTpAloneVocab = 49152;

hipError_t launch_sample_top_p(const TopPArgs& a, hipStream_t st) {
  if (a.rows == 0) return hipSuccess;
  // Where every row has a CU of an MI355X for itself, its list may take all of the LDS: half of a row of 152064 fits, not a seventh, and
  // wider nuclei are found without counting whole rows (256 x 152064, top_p 0.95: sigma 3 at T 1.3 56.5 -> 50.9 us, sigma 2 56.8 ->
  // 53.0; 1 row 49.9 -> 44.8; 46.1, 50.9 and 40.5 if their groups' masses, too, came from such lists, but then what they draw
  // at the edge of an interval would depend on the number of rows).  In shorter rows the smaller list takes as much as is ever worth it, and three rows a
  // CU are no slower alone (32003: 19.4 and 19.7 us).
  // Odd rows (of an odd vocabulary every second one): shifted into place from dwords, or loaded where they start, us: 2000 rows of
  // 152067 201 and 247, 128001 171 and 207, 100003 141 and 168, 32003 64.3 and 67.7; 64 of 32003 16.1 and 17.3.  Rows
  // alone on a CU wait for their vector ALU, which the shift adds to: 64 of 128001 32.4 and 31.4, 152067 35.3 and 35.2.  A row
  // alone that starts on a dword has nothing to shift, and few groups of few rows are not worth the longer code: one of 32003 16.5 and
  // 16.0, 64 of 8193 15.0 and 14.7, of 12291 15.3 and 15.3, of 16385 16.0 and 16.2; 300 of 2051 16.8 and 16.6, of 4099 16.9 and
  // 16.9, of 10243 18.0 and 18.3.
  const bool alone = a.rows <= 256 && a.vocab > kTpAloneVocab;
  const bool odd = ((a.rows > 1 && a.vocab % 2 != 0) || reinterpret_cast<uintptr_t>(a.logits) % 4 != 0) &&
                   a.vocab > (a.rows > 256 ? 4096 : 12288);
  const auto kernel = alone ? sample_top_p_alone_kernel : odd ? sample_top_p_odd_kernel : sample_top_p_kernel;
  hipLaunchKernelGGL(kernel, dim3((unsigned)a.rows), dim3(kTpThreads), 0, st, a);
  return hipGetLastError();
}

// Waves of a workgroup that takes a row whole, 0 where rows are divided between workgroups and a second launch draws.
// Rows of up to 7 chunks (8 up to 512 rows) are taken whole at any number: the second launch is much of the call (30 rows x
// 20481: 7.5 us divided, 6.8 whole; 64 x 32000 7.4 and 6.5; 300 x 32000 10.1 and 9.1).  Longer rows are divided where the
// last round of them over the 256 CUs of an MI355X would leave too many CUs idle (64 x 152064: 10.8 us divided, 16.5 whole, 300: 24.0 and
// 27.3; 100 x 65536 8.2 and 8.3), and whole where they fill it but for a few per cent (256 x 152064: 21.2 and 18.9, 512
// 35.5 and 30.3, 2048 112.5 and 107.1).  Rows that are not aligned to 16 bytes need
// more requests, which few waves on a CU wait longer for: they have to fill it all but exactly, and three rounds of them are
// never as fast (496 x 140001: 33.2 and 35.7, 1000: 61.1 and 64.9, 768: 49.4 and 52.2; 1024 x 40001: 33.5 and 23.4).  As many
// waves as there are chunks, or as a CU has room for (256 x 152064: 8 take 19.1, 4 22.1); fewer of more rows, whose ends
// then overlap (512 x 152064: 8 waves 32.0, 4 30.3, 512 x 100000 24.3 and 21.9; 2048 x 32000 31.8 and 27.2; 768 x 40001 25.4 and 19.4).
// Over 400 sizes of more than 8 chunks that it takes whole, most of them at its edges, calls are 1.105 times as fast as divided; 11 lose
// more than 2 %, the worst of them 4.4 (1845 x 256000: 161 us, divided 154) and 13 (254 x 140001: 22.0, 19.1).
static int sample_row_waves(int rows, int chunks, bool aligned) {
  const int rounds = (rows + 255) / 256;
  if (chunks < 8 || (chunks == 8 && rows <= 512)) return std::min(chunks, rows <= 512 ? 8 : 4);
  const long least = rounds > 4 ? 90 : aligned ? 93 : 99;   // per cent of the CUs' rounds
  if (chunks > kRowMaxChunks || 100l * rows < least * 256l * rounds || (!aligned && rounds == 3)) return 0;
  return rounds == 1 ? kRowMaxWaves : 4;
}

hipError_t launch_sample(const SampleArgs& a, hipStream_t st) {
  if (a.rows == 0) return hipSuccess;
  const bool aligned = a.vocab % 8 == 0 && reinterpret_cast<uintptr_t>(a.logits) % 16 == 0;
  if (const int waves = sample_row_waves(a.rows, a.num_chunks, aligned)) {
    // (More waves on a CU instead of a chunk ahead: 1024 x 65536 29.0 -> 25.9 us, 2048 x 152064 113.2 -> 108.2, 1604 x 20481 23.3 ->
    // 21.3; no slower where there are few.)
    if (waves <= 4) hipLaunchKernelGGL(sample_many_rows_kernel, dim3((unsigned)a.rows), dim3(waves * 64), 0, st, a);
    else hipLaunchKernelGGL(sample_rows_kernel, dim3((unsigned)a.rows), dim3(waves * 64), 0, st, a);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(sample_scan_kernel, dim3((unsigned)a.rows * a.groups_per_row), dim3(256), 0, st, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(sample_pick_kernel, dim3(a.rows), dim3(64), 0, st, a);
  return hipGetLastError();
}

}  // namespace marl
