// Per-token log-probability: out[r] = x[r, tok_r]/T - log sum_v exp(x[r, v]/T), the quantity
// GRPO training (which the paper uses, Section 8.1) consumes for every generated token.
// One streaming pass over the row's bf16 logits with a running (max, sum of exponentials)
// per lane, in base-2 units: y = x * log2(e)/T.  Lanes are combined inside the vector ALU (DPP
// row operations and the row-swap instructions), waves through LDS.  A row is cut into `slices` vocabulary slices when there are too few rows to
// fill the GPU; a small second kernel then combines the slices.
#include "marl_internal.h"
#include "wave_ops.h"

namespace marl {
namespace {

constexpr int kUnroll = 4;

struct MaxSum {
  float m, s;
};

__device__ __forceinline__ float ex2(float x) { return __builtin_amdgcn_exp2f(x); }

// exp2(a - b) that is 0 (not NaN) when a is -inf, whatever b is
__device__ __forceinline__ float ex2_diff(float a, float b) {
  return ex2(a - (b == -INFINITY ? 0.f : b));
}

__device__ __forceinline__ MaxSum combine(MaxSum a, MaxSum b) {
  const float m = fmaxf(a.m, b.m);
  return MaxSum{m, a.s * ex2_diff(a.m, m) + b.s * ex2_diff(b.m, m)};
}

__device__ __forceinline__ void add_one(MaxSum& st, float y) {
  const float m = fmaxf(st.m, y);
  st.s = st.s * ex2_diff(st.m, m) + ex2_diff(y, m);
  st.m = m;
}

// c > 0 (it is log2(e) / T), so the max of the scaled values is the scaled max of the raw ones:
// the scale is applied once to the max and folded into the exponent's fma for the rest.
__device__ __forceinline__ void add_vec(MaxSum& st, u32x4 v, float c) {
  float x[8];
#pragma unroll
  for (int d = 0; d < 4; ++d) {
    x[2 * d] = __uint_as_float(v[d] << 16);
    x[2 * d + 1] = __uint_as_float(v[d] & 0xffff0000u);
  }
  const float x8 = fmaxf(fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3])), fmaxf(fmaxf(x[4], x[5]), fmaxf(x[6], x[7])));
  const float m = fmaxf(st.m, x8 * c);
  const float ms = (m == -INFINITY) ? 0.f : m;
  float sum = 0.f;
#pragma unroll
  for (int e = 0; e < 8; ++e) sum += ex2(__builtin_fmaf(x[e], c, -ms));
  st.s = st.s * ex2(st.m - ms) + sum;
  st.m = m;
}

// (max, sum) of the wave in every lane: the maximum first, then the sums rescaled to it; both
// reductions have a fixed order, so reruns are bit-identical
__device__ __forceinline__ MaxSum wave_combine(MaxSum v) {
  const float m = wave_allreduce(v.m, [](float x, float y) { return fmaxf(x, y); });
  const float s = wave_allreduce(v.s * ex2_diff(v.m, m), [](float x, float y) { return x + y; });
  return MaxSum{m, s};
}

__device__ __forceinline__ float bf16_at(const uint16_t* p) { return __uint_as_float((uint32_t)(*p) << 16); }

// A row's token and its logit are two dependent reads: both are made before the sums are added up, not after.
struct RowToken {
  float x;
  bool valid;
};
__device__ __forceinline__ RowToken read_logit(const LogprobArgs& a, int row, int tok) {
  const bool valid = (unsigned)tok < (unsigned)a.vocab;
  return RowToken{bf16_at(a.logits + (size_t)row * a.vocab + (valid ? tok : 0)), valid};
}
__device__ __forceinline__ float finish_row(const LogprobArgs& a, RowToken t, float m, double sum) {
  return t.valid ? logprob_of(t.x, a.inv_temp_log2e, m, sum) : __uint_as_float(0x7fc00000u);
}

// What bounds it: the read, from about 512 long rows on (2048 x 152064: 92 us, 6.75 TB/s); short rows and few of them
// are a chain of latencies, so the row's token and its logit are read first, what is left of a row behind the
// unrolled loop is requested together, and the waves' sums are independent terms.  (333 x 20481: 6.0 -> 5.2 us,
// 2048 x 20481 20.5 -> 15.3, 2048 x 4096 10.2 -> 5.2, 128 x 152064 12.5 -> 10.0, with the numbers of threads at launch_logprobs.)
template <int kLpThreads>
__global__ __launch_bounds__(kLpThreads) void logprob_kernel(LogprobArgs a) {
  __shared__ MaxSum red[kLpThreads / 64];
  const int row = blockIdx.x / a.slices;
  const int slice = blockIdx.x % a.slices;
  const int tid = threadIdx.x;
  const float c = a.inv_temp_log2e;
  const long v0 = (long)slice * a.slice_len;
  const long v1 = min((long)a.vocab, v0 + a.slice_len);
  const uint16_t* x = a.logits + (size_t)row * a.vocab;
  const bool whole = a.slices == 1;
  const int tok = whole ? ld_uniform(a.tokens + row) : 0;
  RowToken token{0.f, false};
  MaxSum st{-INFINITY, 0.f};

  if (v0 < v1) {
    // elements before the first 16-byte boundary, then whole 16-byte vectors, then the rest
    const uintptr_t addr = reinterpret_cast<uintptr_t>(x + v0);
    const long head = min(v1 - v0, (long)(((16 - (addr & 15)) & 15) >> 1));
    const long b0 = v0 + head;
    const long nvec = (v1 - b0) >> 3;
    const u32x4* xv = reinterpret_cast<const u32x4*>(x + b0);
    const long t0 = b0 + (nvec << 3);
    const long ends = head + (v1 - t0);   // at most 14 elements, one a thread
    const float end = tid < ends ? bf16_at(x + (tid < head ? v0 + tid : t0 + (tid - head))) : -INFINITY;
    long k = tid;
    for (; k + (kUnroll - 1) * kLpThreads < nvec; k += kUnroll * kLpThreads) {
      u32x4 v[kUnroll];
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) v[u] = __builtin_nontemporal_load(xv + k + u * kLpThreads);
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) add_vec(st, v[u], c);
    }
    // what is left, requested together as well (short rows have nothing else)
    u32x4 v[kUnroll - 1];
#pragma unroll
    for (int u = 0; u < kUnroll - 1; ++u) {
      v[u] = u32x4{0xff80ff80u, 0xff80ff80u, 0xff80ff80u, 0xff80ff80u};   // -inf
      if (k + u * kLpThreads < nvec) v[u] = __builtin_nontemporal_load(xv + k + u * kLpThreads);
    }
    if (whole) token = read_logit(a, row, tok);   // (here, so that no row waits for its token before it is read)
#pragma unroll
    for (int u = 0; u < kUnroll - 1; ++u)
      if (__builtin_amdgcn_ballot_w64(k + u * kLpThreads < nvec) != 0) add_vec(st, v[u], c);
    if (tid < ends) add_one(st, end * c);
  }

  st = wave_combine(st);
  if ((tid & 63) == 0) red[tid >> 6] = st;
  __syncthreads();
  if (tid == 0) {   // (independent terms, added in wave order in 64 bits)
    float m = red[0].m;
#pragma unroll
    for (int w = 1; w < kLpThreads / 64; ++w) m = fmaxf(m, red[w].m);
    double sum = 0.0;
#pragma unroll
    for (int w = 0; w < kLpThreads / 64; ++w) sum += (double)(red[w].s * ex2_diff(red[w].m, m));
    if (whole) a.out[row] = finish_row(a, token, m, sum);
    else a.partials[(size_t)row * a.slices + slice] = make_float2(m, (float)sum);
  }
}

// one wave per row: combines the slices in a fixed order
__global__ __launch_bounds__(64) void logprob_finish_kernel(LogprobArgs a) {
  const int row = blockIdx.x;
  const int lane = threadIdx.x;
  const RowToken token = read_logit(a, row, ld_uniform(a.tokens + row));
  MaxSum st{-INFINITY, 0.f};
  for (int k = lane; k < a.slices; k += 64) {
    const float2 p = a.partials[(size_t)row * a.slices + k];
    st = combine(st, MaxSum{p.x, p.y});
  }
  st = wave_combine(st);
  if (lane == 0) a.out[row] = finish_row(a, token, st.m, (double)st.s);
}

}  // namespace

hipError_t launch_logprobs(const LogprobArgs& a, hipStream_t st) {
  if (a.rows == 0) return hipSuccess;
  // Long whole rows: 1024 threads (2048 x 152064: 92.3 us, 92.7 and 93.6 with 512 and 256).  Short rows and slices take
  // less of a workgroup, and smaller ones share a CU (2048 x 20481: 19.6, 15.3, 14.5; 2048 x 4096: 9.6, 6.3, 5.2; 256 x 100003
  // in slices: 13.4, 11.4, 12.0; 256 x 65536 whole: 6.9, 7.7, 10.3).
  const dim3 grid((unsigned)a.rows * a.slices);
  if (a.slice_len <= 8192 && a.slices == 1) hipLaunchKernelGGL(logprob_kernel<256>, grid, dim3(256), 0, st, a);
  else if (a.slice_len <= 49152 || a.slices > 1) hipLaunchKernelGGL(logprob_kernel<512>, grid, dim3(512), 0, st, a);
  else hipLaunchKernelGGL(logprob_kernel<1024>, grid, dim3(1024), 0, st, a);
  return hipGetLastError();
}
hipError_t launch_logprobs_finish(const LogprobArgs& a, hipStream_t st) {
  if (a.rows == 0 || a.slices == 1) return hipSuccess;
  hipLaunchKernelGGL(logprob_finish_kernel, dim3(a.rows), dim3(64), 0, st, a);
  return hipGetLastError();
}

}  // namespace marl
