// a2: Bayesian path saliency (Sec. 3.2.3; App. B.1 Eq. 2).
//
// Kernel 1 (HBM-bound, one workgroup per scored logit row, or per piece of one) streams the row once and stores the
// maximum m and the sum of exp(x - m) with one plain store.  It touches no atomic: a workgroup is not retired before its
// memory operations are acknowledged, and a device-scope atomic takes microseconds to come back while HBM is saturated
// (measured: 16 to 42 us per launch, whether the kernel waits for its atomics or not).
// Kernel 2 merges a row's pieces in order, lp = x[target] - logsumexp(x) as 64-bit fixed point (2^-36 units), and adds up
// the rows of each path.  Integer addition is associative, so the sum does not depend on an order and equal inputs give
// bit-identical scores; a row whose lp is not finite becomes a flag bit instead.
//   scan: one workgroup per path slot reads the path of every row and sums the rows that are its own;
//   atomic, where slots times rows would be too much to read: one thread per row, integer atomics per slot, and a counter
//   that finds the workgroup that finishes last; it turns the sums into scores and puts every accumulator back to zero,
//   the state the next launch expects.
#include <algorithm>
#include <mutex>
#include <type_traits>

#include "sp_device.h"
#include "sp_internal.h"

namespace sp {

constexpr int kSalThreads = 256;
constexpr int kSalUnroll = 4;      // 16-byte vectors in flight per thread and step
constexpr int kSalPieceVecs = kSalThreads * kSalUnroll;          // shortest piece of a row: one step of a workgroup
constexpr double kFixOne = 68719476736.0;        // 2^36
constexpr float kFixLimit = 6.0e7f;              // |lp| above this (about 2^26) is treated as infinite

// Scratch of the entry point that allocates nothing: the launch counter, the per-slot accumulators and
// the per-row partial sums of the largest problem it accepts (kSalStaticRows rows, kSalStaticSlots path slots), on every
// GPU the library runs on; zero at load, and the accumulators are left at zero by every launch.
static __device__ __align__(256) unsigned char scratch[kSalStaticBytes];

template <typename T>
__global__ __launch_bounds__(kSalThreads) void saliency_kernel(const T *__restrict__ logits, int64_t vocab,
                                                             int64_t row_stride,
                                                             const int32_t *__restrict__ target, int n_pieces,
                                                             bool tail_at_once, RowPart *__restrict__ out) {
  constexpr int EV = Elem<T>::kVec;
  const int64_t r = n_pieces == 1 ? blockIdx.x : blockIdx.x / unsigned(n_pieces);
  const int piece = int(blockIdx.x - r * n_pieces);
  const int32_t tgt = target[r];
  __shared__ float sm[kSalThreads / 64], ss[kSalThreads / 64];
  float m = kNegBig, s = 0.f;
  const T *row = logits + r * row_stride;
  if (tgt >= 0) {                                // a row that is not scored does not touch its logits
    const int64_t n_vec = vocab / EV;
    const int64_t v0 = n_pieces == 1 ? 0 : n_vec * piece / n_pieces;
    const int64_t v1 = n_pieces == 1 ? n_vec : n_vec * (piece + 1) / n_pieces;
    const u32x4 *vrow = reinterpret_cast<const u32x4 *>(row);
    // running maximum m (natural units) and s = sum exp(x - m), per thread
    auto step = [&](const u32x4 *raw, auto vectors) {
      constexpr int N = decltype(vectors)::value;
      float x[N * EV];
#pragma unroll
      for (int u = 0; u < N; ++u) Elem<T>::unpack(raw[u], x + u * EV);
      float mx = x[0];
#pragma unroll
      for (int j = 1; j < N * EV; ++j) mx = fmaxf(mx, x[j]);
      const float m_new = fmaxf(m, mx);
      const float mb = m_new * kLog2e;
      float a = 0.f;
#pragma unroll
      for (int j = 0; j < N * EV; ++j) a += fast_exp2(fmaf(x[j], kLog2e, -mb));
      s = fmaf(s, fast_exp2((m - m_new) * kLog2e), a);
      m = m_new;
    };
    int64_t i = v0 + threadIdx.x;
    u32x4 raw[kSalUnroll];
    // whole steps: as many as every lane has, or as many as this lane has
    const int64_t steps_end = tail_at_once ? v1 - (kSalThreads - 1) + threadIdx.x : v1;
    for (; i + (kSalUnroll - 1) * kSalThreads < steps_end; i += kSalPieceVecs) {
#pragma unroll
      for (int u = 0; u < kSalUnroll; ++u) raw[u] = ld16_stream(vrow + i + u * kSalThreads);
      step(raw, std::integral_constant<int, kSalUnroll>{});
    }
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    if (tail_at_once) {
      // A wave requests all that it still has together; where a lane has no vector it takes -inf.
      const int left = __builtin_amdgcn_readfirstlane(int(v1 - i));
      const uint32_t none = EV == 8 ? 0xff80ff80u : 0xff800000u;
      auto last = [&](auto vectors) {
        constexpr int N = decltype(vectors)::value;
#pragma unroll
        for (int u = 0; u < N; ++u) {
          raw[u] = u32x4{none, none, none, none};
          if (lane + u * kSalThreads < left) raw[u] = ld16_stream(vrow + i + u * kSalThreads);
        }
        step(raw, vectors);
      };
      if (left > 3 * kSalThreads) last(std::integral_constant<int, 4>{});
      else if (left > 2 * kSalThreads) last(std::integral_constant<int, 3>{});
      else if (left > kSalThreads) last(std::integral_constant<int, 2>{});
      else if (left > 0) last(std::integral_constant<int, 1>{});
    } else {
      for (; i < v1; i += kSalThreads) {
        raw[0] = ld16(vrow + i);
        step(raw, std::integral_constant<int, 1>{});
      }
    }
    if (piece == n_pieces - 1) {                   // scalar tail (vocab not a multiple of the vector)
      const int64_t j = n_vec * EV + threadIdx.x;
      if (j < vocab) {
        const float x = Elem<T>::load1(row + j);
        const float m_new = fmaxf(m, x);
        s = fmaf(s, fast_exp2((m - m_new) * kLog2e), fast_exp2((x - m_new) * kLog2e));
        m = m_new;
      }
    }
    // combine (m, s) over the workgroup: fixed butterfly inside a wave, then across the waves
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
      const float m_o = __shfl_xor(m, off), s_o = __shfl_xor(s, off);
      const float m_new = fmaxf(m, m_o);
      s = s * fast_exp2((m - m_new) * kLog2e) + s_o * fast_exp2((m_o - m_new) * kLog2e);
      m = m_new;
    }
    if (lane == 0) { sm[wave] = m; ss[wave] = s; }
  }
  __syncthreads();
  if (threadIdx.x != 0) return;
  if (tgt < 0) { out[blockIdx.x] = RowPart{0.f, 0.f, 0.f, 0u}; return; }
  float M = sm[0];
#pragma unroll
  for (int w = 1; w < kSalThreads / 64; ++w) M = fmaxf(M, sm[w]);
  float S = 0.f;
#pragma unroll
  for (int w = 0; w < kSalThreads / 64; ++w) S += ss[w] * fast_exp2((sm[w] - M) * kLog2e);
  const int64_t t = tgt < vocab ? tgt : vocab - 1;
  out[blockIdx.x] = RowPart{M, S, piece == 0 ? Elem<T>::load1(row + t) : 0.f, 1u};
}

// a row's log-likelihood in fixed point, or flag bits when it is not finite
struct RowLp {
  long long q;
  uint32_t flags, scored;
};
__device__ __forceinline__ RowLp row_lp(const RowPart *__restrict__ part, int64_t r, int n_pieces) {
  const RowPart *p = part + r * n_pieces;
  const RowPart first = p[0];
  RowLp v{0ll, 0u, first.scored};
  if (!first.scored) return v;
  float M = first.m, S = first.s;
  for (int i = 1; i < n_pieces; ++i) {
    const RowPart o = p[i];
    const float m_new = fmaxf(M, o.m);
    S = S * fast_exp2((M - m_new) * kLog2e) + o.s * fast_exp2((o.m - m_new) * kLog2e);
    M = m_new;
  }
  const float lp = first.x_target - (M + __logf(S));
  if (lp != lp || fabsf(lp) > kFixLimit) v.flags = lp != lp ? 4u : (lp < 0.f ? 1u : 2u);
  else v.q = __double2ll_rn(double(lp) * kFixOne);
  return v;
}
__device__ __forceinline__ float slot_score(long long sum, uint32_t count, uint32_t flags, int mode, const float *prior,
                                            int64_t slot) {
  float x = float(double(sum) * (1.0 / kFixOne));
  if (flags) x = ((flags & 4u) || (flags & 3u) == 3u) ? __builtin_nanf("") : ((flags & 1u) ? -INFINITY : INFINITY);
  if (mode == 1) x = count > 0 ? x / float(count) : 0.f;
  if (prior) x += prior[slot];
  return x;
}
__device__ __forceinline__ int32_t clamp_slot(int32_t slot, int32_t n_slots) {
  return slot < 0 ? 0 : (slot >= n_slots ? n_slots - 1 : slot);
}

constexpr int kRedThreads = 256;
constexpr int64_t kScanWideRows = 9 * 256, kScanWideSlots = 256;   // a scan of 1024 threads, see the launch
constexpr int64_t kScanReads = int64_t(1) << 22, kScanRows = 4096, kScanRowsManySlots = 7168, kManySlots = 500;
// One workgroup per slot.  Bound by the latency of two dependent reads (row_path, then the slot's rows); there is no atomic,
// and the reads of row_path are independent of each other and come from the L2.  340 rows of 20 slots: 3.8 us (the atomic
// kernel 6.2), 3840 rows of 160 slots: 4.7 us (6.1) with 256 threads.  NT: a thread has eight reads in flight, see the launch.
template <int NT>
__global__ __launch_bounds__(NT) void saliency_scan_kernel(const RowPart *__restrict__ part, int n_pieces,
                                                                    const int32_t *__restrict__ row_path, int32_t n_rows,
                                                                    const float *__restrict__ prior, int32_t n_slots,
                                                                    int mode, float *__restrict__ score) {
  constexpr int U = 8;
  const int32_t mine = blockIdx.x;
  long long q = 0;
  uint32_t count = 0, flags = 0;
  for (int32_t r0 = threadIdx.x; r0 < n_rows; r0 += U * NT) {
    int32_t slot[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int32_t r = r0 + u * NT;
      slot[u] = r < n_rows ? clamp_slot(row_path[r], n_slots) : -1;
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (slot[u] == mine) {
        const RowLp v = row_lp(part, r0 + u * NT, n_pieces);
        q += v.q;
        count += v.scored;
        flags |= v.flags;
      }
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    q += __shfl_xor(q, off);
    count += __shfl_xor(count, off);
    flags |= __shfl_xor(flags, off);
  }
  __shared__ long long s_q[NT / 64];
  __shared__ uint32_t s_c[NT / 64], s_f[NT / 64];
  const int wave = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) { s_q[wave] = q; s_c[wave] = count; s_f[wave] = flags; }
  __syncthreads();
  if (threadIdx.x != 0) return;
#pragma unroll
  for (int w = 1; w < NT / 64; ++w) { q += s_q[w]; count += s_c[w]; flags |= s_f[w]; }
  score[mine] = slot_score(q, count, flags, mode, prior, mine);
}

__global__ __launch_bounds__(kRedThreads) void saliency_reduce_kernel(const RowPart *__restrict__ part, int n_pieces,
                                                                      const int32_t *__restrict__ row_path,
                                                                      int64_t n_rows, const float *__restrict__ prior,
                                                                      int32_t n_slots, int mode, SalSlot *__restrict__ acc,
                                                                      uint32_t *__restrict__ done,
                                                                      float *__restrict__ score) {
  const int64_t r = (int64_t)blockIdx.x * kRedThreads + threadIdx.x;
  __shared__ int s_last;
  RowLp v{0ll, 0u, 0u};
  int32_t slot = 0;
  if (r < n_rows) {
    v = row_lp(part, r, n_pieces);
    slot = clamp_slot(row_path[r], n_slots);
  }
  // Rows of one path usually sit next to each other, and atomics on one address are performed one after
  // the other: a wave first adds up, per slot, what its own lanes hold (up to kWaveSlots different slots),
  // and one lane sends the total.  Lanes left over send their own value.  The atomics return a value that
  // is kept alive: the barrier below is passed only after they have been performed, so the workgroup that
  // reads the last count sees every sum complete.
  constexpr int kWaveSlots = 4;
  const int lane = threadIdx.x & 63;
  unsigned long long pending = __ballot(v.scored != 0u);
  for (int it = 0; it < kWaveSlots && pending; ++it) {
    const int lead = __ffsll((long long)pending) - 1;
    const int32_t s0 = __shfl(slot, lead);
    const bool mine = ((pending >> lane) & 1ull) && slot == s0;
    long long q = mine && !v.flags ? v.q : 0ll;
    unsigned cnt = mine ? 1u : 0u, fl = mine ? v.flags : 0u;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
      q += __shfl_xor(q, off);
      cnt += __shfl_xor(cnt, off);
      fl |= __shfl_xor(fl, off);
    }
    if (lane == lead) {
      SalSlot *a = acc + s0;
      unsigned long long r0 = 0;
      unsigned r1 = 0;
      if (q) r0 = __hip_atomic_fetch_add(&a->sum, (unsigned long long)q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (fl) r1 = __hip_atomic_fetch_or(&a->flags, fl, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      const unsigned r2 = __hip_atomic_fetch_add(&a->count, cnt, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      asm volatile("" ::"v"(r0), "v"(r1), "v"(r2) : "memory");
    }
    pending &= ~__ballot(mine);
  }
  if ((pending >> lane) & 1ull) {
    SalSlot *a = acc + slot;
    unsigned long long r0 = 0;
    unsigned r1 = 0;
    if (v.flags) r1 = __hip_atomic_fetch_or(&a->flags, v.flags, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else r0 = __hip_atomic_fetch_add(&a->sum, (unsigned long long)v.q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const unsigned r2 = __hip_atomic_fetch_add(&a->count, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("" ::"v"(r0), "v"(r1), "v"(r2) : "memory");
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    const unsigned before = __hip_atomic_fetch_add(done, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    s_last = before == gridDim.x - 1 ? 1 : 0;
  }
  __syncthreads();
  if (!s_last) return;
  // the last workgroup: sums -> scores, accumulators back to zero
  for (int i = threadIdx.x; i < n_slots; i += kRedThreads) {
    SalSlot *a = acc + i;
    SalSlot v;
    v.sum = __hip_atomic_load(&a->sum, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    v.count = __hip_atomic_load(&a->count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    v.flags = __hip_atomic_load(&a->flags, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    score[i] = slot_score((long long)v.sum, v.count, v.flags, mode, prior, i);
    __hip_atomic_store(&a->sum, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(&a->count, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(&a->flags, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  if (threadIdx.x == 0) __hip_atomic_store(done, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// scratch: the launch counter (256 bytes), one SalSlot per path slot of the capacity, then one RowPart per
// row; the counter and the accumulators are zero before the launch and left at zero.
hipError_t launch_saliency(const void *logits, sp_dtype dt, int64_t n_rows, int64_t vocab, int64_t row_stride,
                           const int32_t *target, const int32_t *row_path, const float *prior, int32_t n_slots,
                           int mode, void *scratch, int32_t cap_slots, float *score, hipStream_t s) {
  uint32_t *done = static_cast<uint32_t *>(scratch);
  SalSlot *acc = reinterpret_cast<SalSlot *>(static_cast<unsigned char *>(scratch) + 256);
  RowPart *part = reinterpret_cast<RowPart *>(acc + cap_slots);
  // With fewer rows than workgroups that the device holds at once (8 per compute unit), rows are cut into as many pieces as
  // fill it, none shorter than one step of a workgroup.  340 fp32 rows of 50257 in 6 pieces: 11.6 us, 5.9 TB/s (whole rows,
  // most compute units with one workgroup's 16 KB in flight: 14.2 us).  More pieces than that do not pay (whole call with
  // top-k, up to 2048 / 4096 / 8192 / 16384 workgroups): 340 rows 19.4 / 20.6 / 20.6 / 20.5 us, 1500 bf16 rows of 50432
  // 32.5 / 32.1 / 36.5 / 34.6, 3840 of them 68.3 / 68.4 / 68.7 / 71.4.
  const int64_t n_vec = vocab / (dt == SP_BF16 ? 8 : 4);
  int n_pieces = 1;
  if (n_rows > 0)
    n_pieces = int(std::max<int64_t>(1, std::min(kSalSplitRows / n_rows, n_vec / kSalPieceVecs)));
  // The last vectors of a row (or piece) at once, except where thousands of rows keep every compute unit busy with others:
  // us a call, all at once / one after the other, 4000 bf16 rows of 6200 17.6 / 19.8, 4097 fp32 rows of 32000 83.8 / 86.5;
  // 5000 bf16 rows of 128256 203.8 / 201.8, 20000 of 32000 197.5 / 192.9, 20000 of 2048 31.4 / 28.5.
  const bool tail_at_once = n_rows <= kScanRows;
  if (n_rows > 0) {
    const dim3 grid(unsigned(n_rows * n_pieces));
    if (dt == SP_BF16)
      hipLaunchKernelGGL(saliency_kernel<__bf16>, grid, dim3(kSalThreads), 0, s, static_cast<const __bf16 *>(logits),
                         vocab, row_stride, target, n_pieces, tail_at_once, part);
    else
      hipLaunchKernelGGL(saliency_kernel<float>, grid, dim3(kSalThreads), 0, s, static_cast<const float *>(logits), vocab,
                         row_stride, target, n_pieces, tail_at_once, part);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  // The scan reads rows * slots path numbers from the L2, and a thread of it every 256th row.  Measured, us a call of 512
  // fp32 logits a row, scan / atomics: 3000 rows of 20 slots 9.2 / 9.4; 4096 rows of 500 slots 10.5 / 14.6; 4097 of 20
  // 11.0 / 10.3, of 500 11.2 / 15.2; 6500 of 600 14.9 / 16.7, of 20 14.4 / 12.4; 8192 of 512 16.6 / 16.6, of 100 16.2 / 14.4.
  // kScanReads are 16 MB over all workgroups.  The scan launches a workgroup per slot, whatever the rows, so it bounds the
  // slots as well (a launch ends at 2^24 workgroups).
  if (n_rows <= (n_slots >= kManySlots ? kScanRowsManySlots : kScanRows) &&
      std::max<int64_t>(n_rows, 1) * n_slots <= kScanReads) {
    // A thread has eight reads of row_path in flight.  With 256 threads more rows than 2048 take a second round of them, each
    // a memory latency, and 1024 threads one; but a workgroup of 1024 leaves room for one other on a compute unit, so many
    // slots wait for places.  us a call of 512 bf16 logits a row, 256 / 1024 threads: 2049 rows of 20 slots 8.0 / 8.3, 2500 of
    // 160 8.7 / 8.45, 3000 of 20 9.2 / 8.6, 4096 of 100 10.3 / 9.5, 4096 of 500 10.6 / 10.65, 4096 of 1000 11.2 / 13.4, 3000 of
    // 1300 10.3 / 14.7; 3840 rows of 50432 logits and 160 slots 62.7 / 61.7, with top-k 67.1 / 65.9.
    auto scan = [&](auto threads) {
      constexpr int NT = decltype(threads)::value;
      hipLaunchKernelGGL(saliency_scan_kernel<NT>, dim3(unsigned(n_slots)), dim3(NT), 0, s, part, n_pieces, row_path,
                         int32_t(n_rows), prior, n_slots, mode, score);
    };
    if (n_rows > kScanWideRows && n_slots <= kScanWideSlots) scan(std::integral_constant<int, 1024>{});
    else scan(std::integral_constant<int, 256>{});
    return hipGetLastError();
  }
  const unsigned grid = n_rows > 0 ? unsigned((n_rows + kRedThreads - 1) / kRedThreads) : 1u;
  hipLaunchKernelGGL(saliency_reduce_kernel, dim3(grid), dim3(kRedThreads), 0, s, part, n_pieces, row_path, n_rows, prior,
                     n_slots, mode, acc, done, score);
  return hipGetLastError();
}

// Address of this device's copy of the static scratch array.  In host code the array's name is only a
// stand-in, not a device address: the address comes from the runtime, once per device, with that device
// current (the caller has made it current), and is kept per device.
hipError_t saliency_static_scratch(int device, void **out) {
  static std::mutex mu;
  static void *ptrs[kMaxDevices] = {};
  if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(mu);
  if (!ptrs[device]) {
    void *p = nullptr;
    hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    ptrs[device] = p;
  }
  *out = ptrs[device];
  return hipSuccess;
}

}  // namespace sp
