// a3: greedy top-k of the per-path posterior (Sec. 3.2.3; Alg. 3).  One workgroup per prompt.
// Each path's rank is the number of paths that come before it in the order
// (score descending, index ascending, NaN last); paths with rank < k write kept[rank].
#include "sp_internal.h"

namespace sp {

// Place of a score in the order as one number, larger = earlier: the float's bits made monotone (NaN lowest, -0 as +0),
// then the lower index first.
__device__ __forceinline__ uint64_t order_key(float x, int i) {
  const uint32_t u = __float_as_uint(x + 0.f);
  const uint32_t k = x != x ? 0u : (u >> 31) ? ~u : u | 0x80000000u;
  return (uint64_t(k) << 32) | uint32_t(~i);
}

// Bound by latency (path_off, scores, the ranking loop): one comparison of 64-bit keys per pair, so the loop is unrolled
// and its LDS reads are in flight together.  20 scores: about 1.8 us less than a
// loop that compares scores and tells ties and NaN apart one by one (saliency and top-k of one prompt 20.4 -> 18.7 us).
__global__ __launch_bounds__(256) void topk_kernel(const float *__restrict__ score,
                                                   const int32_t *__restrict__ path_off, int32_t k,
                                                   int32_t n_cap, int32_t *__restrict__ kept) {
  extern __shared__ uint64_t s_key[];
  const int b = blockIdx.x;
  const int base = path_off[b];
  int n = path_off[b + 1] - base;
  n = n < 0 ? 0 : n;
  // a prompt with more paths than the caller's bound is still ranked completely: its scores are then
  // read from global memory instead of the LDS copy (slower, never truncated)
  const bool staged = n <= n_cap;
  const float *sc = score + base;
  if (staged)
    for (int i = threadIdx.x; i < n; i += blockDim.x) s_key[i] = order_key(sc[i], i);
  for (int j = n + threadIdx.x; j < k; j += blockDim.x) kept[(int64_t)b * k + j] = -1;
  __syncthreads();
  for (int i = threadIdx.x; i < n; i += blockDim.x) {
    int rank = 0;
    if (staged) {
      const uint64_t mine = s_key[i];
#pragma unroll 8
      for (int j = 0; j < n; ++j) rank += s_key[j] > mine ? 1 : 0;
    } else {
      const uint64_t mine = order_key(sc[i], i);
      for (int j = 0; j < n; ++j) rank += order_key(sc[j], j) > mine ? 1 : 0;
    }
    if (rank < k) kept[(int64_t)b * k + rank] = i;
  }
}

hipError_t launch_topk(const float *score, const int32_t *path_off, int32_t n_prompts, int32_t n_paths_max,
                       int32_t k, int32_t *kept, hipStream_t s) {
  hipLaunchKernelGGL(topk_kernel, dim3(n_prompts), dim3(256), size_t(n_paths_max) * sizeof(uint64_t), s, score,
                     path_off, k, n_paths_max, kept);
  return hipGetLastError();
}

}  // namespace sp
