// a4: single-token decode attention over the joined cache (Sec. 3.2.3; Alg. 3 generation loop).
//
// The kept paths' caches are "simply concatenated" in the paper; here nothing is copied: each
// workgroup resolves the concatenation [shared; kept path 0; ...; kept path k-1; response; new]
// through the plan's range tables and the device-resident kept table, and streams K and V rows
// straight from the packed prefill cache.  HBM-bound: every K/V byte is read once per step.
//
// Workgroup = (prompt, KV head, chunk of GC query heads, piece of the key list), 256 threads.
// The key list is cut into n_pieces equal pieces.  With many prompts one piece is enough to fill the
// chip; a few prompts leave most compute units idle and every workgroup alone with a long serial
// stream (a compute unit takes ~16 B/clk from memory whatever it does), so there each piece gets a
// workgroup of its own and the workgroup that finishes last merges the pieces in their order.
// decode_pieces() below states the rule and what it measured; a launch for one prompt of 32 heads with 370 keys goes
// from 16.0 to 8.4 us, one for six prompts of 32/8 heads with ~820 keys from 50 to 11 us.  What is left of a small
// launch is a chain of latencies (us): tables 1.3, K/V loads and arithmetic 2.5, sum over the waves 0.5, storing the
// piece and counting in 0.8, merge 1.2.
//
// Two ways to compute a piece:
//   decode_kernel      one query head per K/V row group, or fp32: a key row is covered by LPK lanes with one
//                      16-byte load each, dot products on the vector unit, reduced over the lanes;
//   decode_gqa_kernel  bf16 with 2..8 query heads per KV head: the products with K run on the matrix cores
//                      (a tile of 16 keys times up to 16 heads), which takes the per-head lane reductions
//                      away; the weighted sum of V stays on the vector unit with P in fp32.
#include <algorithm>
#include <type_traits>

#include "sp_device.h"
#include "sp_internal.h"

namespace sp {

constexpr int kDecThreads = 256;
constexpr int kDecWaves = kDecThreads / 64;
constexpr int kDecMaxRanges = 128;
constexpr int kDecUnroll = 4;

struct DecodeDev {
  const int32_t *kept;
  int32_t k;
  const void *Kp, *Vp;
  int64_t kv_tok_stride, kv_head_stride;
  void *Kr, *Vr;
  float *pos_resp;
  int32_t resp_capacity;
  const int32_t *resp_len;
  int32_t resp_len_add;
  const float *new_pos;
  const void *q_new, *k_new, *v_new;
  void *o_out;
  float scale;
  int32_t n_pieces;        // pieces of the key list
  int32_t pieces_per_wg;   // n_pieces (one workgroup does them all, in order) or 1
  float *part;             // with one workgroup per piece: [row][piece][D] sums, then [row][piece] {max, sum}
  uint32_t *count;         // and one arrival counter per (prompt, KV head, chunk of query heads), zero between launches
  int32_t chunks_together; // see my_share
  int32_t few_wgs;         // see build_key_table
};

// The key list of one (prompt, KV head) as ranges with running key counts, in LDS: the prefill ranges of the
// shared part and of the kept paths, the response cache, the new token.
struct KeyTable {
  int32_t cum[kDecMaxRanges + 3];
  int64_t stride[kDecMaxRanges + 2];           // bytes from one token to the next
  const char *k[kDecMaxRanges + 2], *v[kDecMaxRanges + 2];
  const float *pos[kDecMaxRanges + 2];
  int32_t s_cnt[kDecMaxRanges], s_keys[kDecMaxRanges];
  int32_t n_total, n_ranges;
};

// One thread per source follows the tables (kept -> path slot descriptor, which carries the first range), so the
// dependent loads of all sources run side by side; a prefix over the sources puts the ranges in order.
// Where no prompt has more than 64 paths, the descriptors of a prompt's paths lie at a fixed place (path_stride; upload_plan
// says where not) and the first wave reads all of them while `kept` is on its way, and picks from its lanes: one memory latency less for every
// launch, and no barrier between the two halves, which one wave does (four tokens of six prompts of 32/8 heads 47.0 -> 45.1 us,
// a request with five tokens of one prompt of 32 heads 89.1 -> 86.2).  With more than four workgroups to a compute unit the
// others' streams hide the latency, and the reads of paths that are not kept cost 0.2 % (64 prompts, 32 heads: 91.1 / 91.4).
template <typename T, int D>
__device__ __forceinline__ void build_key_table(const PlanDev &pd, const DecodeDev &a, int b, int g, int len_r, bool bias,
                                                KeyTable &t) {
  const int tid = threadIdx.x, Hkv = pd.n_kv_heads;
  const int n_src = min(a.k, kDecMaxRanges - 1) + 1;      // k beyond that: prompts without paths, nothing to keep
  const bool one_wave = a.few_wgs && pd.path_stride > 0 && n_src <= 64;
  RangeDesc src{0, 0, 0, 0};
  if (one_wave) {
    if (tid < 64) {
      RangeDesc path{0, 0, 0, 0};
      int kp = -1;
      if (tid < pd.path_stride) path = pd.path_desc[b * pd.path_stride + tid];
      if (tid > 0 && tid < n_src) kp = a.kept[(int64_t)b * a.k + (tid - 1)];
      const RangeDesc shared = pd.shared_desc[b];
      const RangeDesc mine{__shfl(path.beg, kp & 63), __shfl(path.end, kp & 63), __shfl(path.tok_start, kp & 63),
                           __shfl(path.len, kp & 63)};
      if (tid == 0) src = shared;
      else if (kp >= 0 && kp < pd.path_stride) src = mine;   // paths that the prompt does not have are empty
    }
  } else if (tid == 0) {
    src = pd.shared_desc[b];
  } else if (tid < n_src) {
    const int p0 = pd.path_off[b], np = pd.path_off[b + 1] - p0;
    const int kp = a.kept[(int64_t)b * a.k + (tid - 1)];
    if (kp >= 0 && kp < np) src = pd.path_desc[pd.path_stride > 0 ? b * pd.path_stride + kp : p0 + kp];
  }
  const int beg = src.beg, end = src.end;
  if (tid < n_src) {
    int keys = end > beg ? src.len : 0;
    for (int r = beg + 1; r < end; ++r) keys += pd.dec_ranges[r].len;
    t.s_cnt[tid] = end - beg;
    t.s_keys[tid] = keys;
  }
  if (one_wave) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  } else {
    __syncthreads();
  }
  if (tid < n_src) {
    int at = 0, cum = 0;
    for (int i = 0; i < tid; ++i) { at += t.s_cnt[i]; cum += t.s_keys[i]; }
    const char *kb = static_cast<const char *>(a.Kp) + (int64_t)g * a.kv_head_stride * int64_t(sizeof(T));
    const char *vb = static_cast<const char *>(a.Vp) + (int64_t)g * a.kv_head_stride * int64_t(sizeof(T));
    const int64_t stride = a.kv_tok_stride * int64_t(sizeof(T));
    for (int r = beg; r < end && at < kDecMaxRanges; ++r, ++at) {
      const KeyRange kr = r == beg ? KeyRange{src.tok_start, src.len} : pd.dec_ranges[r];
      t.cum[at] = cum;
      t.stride[at] = stride;
      t.k[at] = kb + kr.tok_start * stride;
      t.v[at] = vb + kr.tok_start * stride;
      t.pos[at] = bias ? pd.tok_pos + kr.tok_start : nullptr;
      cum += kr.len;
    }
    if (tid == n_src - 1) {
      const int64_t row = int64_t(b) * a.resp_capacity * Hkv + g;
      if (len_r > 0) {
        t.cum[at] = cum;
        t.stride[at] = int64_t(Hkv) * D * int64_t(sizeof(T));
        t.k[at] = reinterpret_cast<const char *>(static_cast<const T *>(a.Kr) + row * D);
        t.v[at] = reinterpret_cast<const char *>(static_cast<const T *>(a.Vr) + row * D);
        t.pos[at] = bias ? a.pos_resp + int64_t(b) * a.resp_capacity : nullptr;
        cum += len_r;
        ++at;
      }
      t.cum[at] = cum;
      t.stride[at] = 0;
      t.k[at] = reinterpret_cast<const char *>(static_cast<const T *>(a.k_new) + ((int64_t)b * Hkv + g) * D);
      t.v[at] = reinterpret_cast<const char *>(static_cast<const T *>(a.v_new) + ((int64_t)b * Hkv + g) * D);
      t.pos[at] = bias ? a.new_pos + b : nullptr;
      t.cum[at + 1] = cum + 1;
      t.n_total = cum + 1;
      t.n_ranges = at + 1;
    }
  }
  __syncthreads();
}

// K, V and positions are read through pointers from the table: see global_ptr
template <bool STREAM>
__device__ __forceinline__ u32x4 ld16_kv(const char *p) {
  if constexpr (STREAM) return __builtin_nontemporal_load(global_ptr<u32x4>(p));
  else return *global_ptr<u32x4>(p);
}

// Range of a key (vk < n_total, so every search ends at the latest on the new token's range).  Every lane keeps one
// running count, so that the range of a wave-uniform key is one comparison and a bit count; walking the counts in LDS
// instead costs a dependent LDS read per range, which a piece of a few dozen keys feels (1 us of 4).
struct RangeSearch {
  const KeyTable &t;
  int32_t my_end;                              // end of range `lane`
  __device__ __forceinline__ explicit RangeSearch(const KeyTable &tab) : t(tab) {
    const int lane = threadIdx.x & 63;
    my_end = lane < t.n_ranges ? t.cum[lane + 1] : INT32_MAX;
  }
  __device__ __forceinline__ int from(int i, int vk) const {
    while (t.cum[i + 1] <= vk) ++i;
    return i;
  }
  // vk wave-uniform
  __device__ __forceinline__ int uniform(int vk) const {
    const int i = __popcll(__ballot(my_end <= vk));
    return i < 64 ? i : __builtin_amdgcn_readfirstlane(from(64, vk));
  }
};

__device__ __forceinline__ int64_t uniform64(int64_t x) {
  const uint32_t lo = __builtin_amdgcn_readfirstlane(uint32_t(x)), hi = __builtin_amdgcn_readfirstlane(uint32_t(x >> 32));
  return int64_t((uint64_t(hi) << 32) | lo);
}

// What a workgroup does: (prompt, KV head) pair and chunk of that head's query heads.  With several chunks (!STREAM) and
// pairs that divide by 8, the chunks of a pair follow each other on one XCD (workgroups go round the 8 XCDs) and find the
// pair's K and V in its L2.  64 fp32 prompts, us with all pairs' first chunk before any second / as here: 28/4 heads (seven
// chunks) 114.5 / 58.9, 36/4 (nine) 150.5 / 70.9, 40/4 (five) 73.8 / 71.7.
struct Share { int pair, chunk; };
template <bool STREAM>
__device__ __forceinline__ Share my_share(const DecodeDev &a) {
  if (STREAM) return {int(blockIdx.x), 0};
  if (a.chunks_together) return {int(blockIdx.z * 8 + blockIdx.x % 8), int(blockIdx.x / 8)};
  return {int(blockIdx.x), int(blockIdx.z)};
}

// rows of the response cache that take part (the new token is not one of them), and the row the new token goes to
struct RespRows { int read, write; };
__device__ __forceinline__ RespRows resp_rows(const DecodeDev &a, int b) {
  const int len_b = (a.resp_len ? a.resp_len[b] : 0) + a.resp_len_add;
  return {len_b < a.resp_capacity ? (len_b < 0 ? 0 : len_b) : a.resp_capacity, len_b};
}

// append the new token's K/V (and position) to the response cache: one workgroup per (prompt, KV head)
template <typename T, int D>
__device__ __forceinline__ void append_new(const PlanDev &pd, const DecodeDev &a, int b, int g, int row) {
  constexpr int EV = Elem<T>::kVec, LPK = D / EV;
  const int Hkv = pd.n_kv_heads, tid = threadIdx.x, sub = tid % LPK;
  if (row < 0 || row >= a.resp_capacity) return;
  const int64_t to = (((int64_t)b * a.resp_capacity + row) * Hkv + g) * D + sub * EV, from = ((int64_t)b * Hkv + g) * D + sub * EV;
  if (tid < LPK) st16(static_cast<T *>(a.Kr) + to, ld16(static_cast<const T *>(a.k_new) + from));
  else if (tid < 2 * LPK) st16(static_cast<T *>(a.Vr) + to, ld16(static_cast<const T *>(a.v_new) + from));
  if (g == 0 && tid == 0 && a.pos_resp && a.new_pos) a.pos_resp[(int64_t)b * a.resp_capacity + row] = a.new_pos[b];
}

// What the key groups of one piece left in LDS: maximum, sum, weighted V sums per group and head.
template <int D, int GC, int NG>
struct GroupSums {
  float m[NG][GC], l[NG][GC];
  float acc[NG][GC][D];
};

// Merge of pieces.  Thread t owns elements t, t + 256, ... of the GC x D outputs.  Pieces are added one after the
// other in their order, whoever computed them: the result does not depend on how the pieces were spread over
// workgroups.
template <int D, int GC>
struct PieceMerge {
  static constexpr int NE = (GC * D + kDecThreads - 1) / kDecThreads;
  float m[NE], num[NE], den[NE];
  __device__ __forceinline__ void init() {
#pragma unroll
    for (int i = 0; i < NE; ++i) { m[i] = kNegBig; num[i] = 0.f; den[i] = 0.f; }
  }
  __device__ __forceinline__ void add(int i, float pm, float pn, float pl) {
    const float mx = fmaxf(m[i], pm), wa = fast_exp2(m[i] - mx), wb = fast_exp2(pm - mx);
    num[i] = num[i] * wa + pn * wb;
    den[i] = den[i] * wa + pl * wb;
    m[i] = mx;
  }
  // element i of the piece whose groups are in LDS
  template <int NG>
  __device__ __forceinline__ void piece(const GroupSums<D, GC, NG> &s, int idx, float &pm, float &pn, float &pl) const {
    const int c = idx / D, e = idx % D;
    pm = s.m[0][c];
#pragma unroll
    for (int j = 1; j < NG; ++j) pm = fmaxf(pm, s.m[j][c]);
    pn = 0.f; pl = 0.f;
#pragma unroll
    for (int j = 0; j < NG; ++j) {
      const float w = fast_exp2(s.m[j][c] - pm);
      pn = fmaf(w, s.acc[j][c][e], pn);
      pl = fmaf(w, s.l[j][c], pl);
    }
  }
};

// Ends a workgroup: after every piece the groups' sums are in `s`.  A workgroup that has all pieces adds them up in
// registers.  With one workgroup per piece, each stores its piece with agent-scope (write-through) stores, waits for
// them and counts itself in; the last one to arrive reads all pieces back, merges them and puts the counter back to
// zero.  There is no device-scope fence on purpose: it would write back and invalidate the whole L2 (measured: 67 us
// for a step), while the stores and loads here bypass it for these few kilobytes alone.
template <typename T, int D, int GC, int NG, class ComputePiece>
__device__ __forceinline__ void run_pieces(const PlanDev &pd, const DecodeDev &a, Share me, int b, int head0, int n_heads,
                                           int n_total, GroupSums<D, GC, NG> &s, ComputePiece &&compute) {
  using PM = PieceMerge<D, GC>;
  const int tid = threadIdx.x, Hq = pd.n_q_heads;
  const int first = a.pieces_per_wg == 1 ? int(blockIdx.y) : 0;
  // pieces are multiples of 16 keys
  const int chunk = ((n_total + a.n_pieces - 1) / a.n_pieces + 15) & ~15;
  PM run;
  run.init();
  for (int p = first; p < first + a.pieces_per_wg; ++p) {
    if (p > first) __syncthreads();                       // the merge below has read the previous piece's sums
    compute(min(p * chunk, n_total), min((p + 1) * chunk, n_total));
    __syncthreads();
#pragma unroll
    for (int i = 0; i < PM::NE; ++i) {
      const int idx = tid + i * kDecThreads;
      if (idx >= GC * D) continue;
      float pm, pn, pl;
      run.piece(s, idx, pm, pn, pl);
      if (a.pieces_per_wg == a.n_pieces) {
        run.add(i, pm, pn, pl);
      } else {
        const int64_t row = ((int64_t)b * Hq + min(head0 + idx / D, Hq - 1)) * a.n_pieces + p;
        const int64_t rows = (int64_t)pd.n_prompts * Hq * a.n_pieces;
        if (idx / D < n_heads) {
          __hip_atomic_store(a.part + row * D + idx % D, pn, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          if (idx % D == 0) {
            __hip_atomic_store(a.part + rows * D + row * 2, pm, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(a.part + rows * D + row * 2 + 1, pl, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          }
        }
      }
    }
  }
  if (a.pieces_per_wg != a.n_pieces) {
    __shared__ int s_last;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // this wave's stores have been performed
    __syncthreads();
    if (tid == 0) {
      uint32_t *ctr = a.count + (me.chunk * pd.n_prompts * pd.n_kv_heads + me.pair);
      const uint32_t before = __hip_atomic_fetch_add(ctr, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      s_last = before == uint32_t(a.n_pieces - 1);
      if (s_last) __hip_atomic_store(ctr, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    if (!s_last) return;
#pragma unroll
    for (int i = 0; i < PM::NE; ++i) {
      const int idx = tid + i * kDecThreads;
      if (idx >= GC * D || idx / D >= n_heads) continue;
      const int64_t row0 = ((int64_t)b * Hq + head0 + idx / D) * a.n_pieces;
      const float *acc = a.part + row0 * D + idx % D, *ml = a.part + (int64_t)pd.n_prompts * Hq * a.n_pieces * D + row0 * 2;
      for (int p0 = 0; p0 < a.n_pieces; p0 += 8) {        // eight pieces' loads in flight
        float pn[8], pm[8], pl[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const int p = min(p0 + j, a.n_pieces - 1);
          pn[j] = __hip_atomic_load(acc + p * D, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          pm[j] = __hip_atomic_load(ml + 2 * p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          pl[j] = __hip_atomic_load(ml + 2 * p + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
#pragma unroll
        for (int j = 0; j < 8; ++j)
          if (p0 + j < a.n_pieces) run.add(i, pm[j], pn[j], pl[j]);
      }
    }
  }
#pragma unroll
  for (int i = 0; i < PM::NE; ++i) {
    const int idx = tid + i * kDecThreads;
    if (idx < GC * D && idx / D < n_heads)
      Elem<T>::store1(static_cast<T *>(a.o_out) + ((int64_t)b * Hq + head0 + idx / D) * D + idx % D, run.num[i] / run.den[i]);
  }
}

// STREAM: a workgroup reads its K and V rows alone (one chunk of query heads per KV head), so they are read non-temporally
// (64 prompts of 32 heads, 430 keys: 103.1 -> 93.0 us, 5.8 TB/s).  Where several chunks read the same rows, cached loads let
// the later ones find them in the caches (64 fp32 prompts of 40/4 heads, five chunks: non-temporally 100.7, cached 77.7 us).
// Four waves per SIMD for one head, except that bf16 with positions does not fit their 128 registers: with three it takes
// 135 and spills none (64 prompts, 32 heads: 101.1 -> 87.5 us; at four, 6 spilled).
template <typename T, int D, int GC, bool BIAS, bool STREAM>
__global__ __launch_bounds__(kDecThreads, GC == 1 ? (BIAS && sizeof(T) == 2 ? 3 : 4) : 2) void decode_kernel(PlanDev pd, DecodeDev a) {
  constexpr int EV = Elem<T>::kVec;       // elements per 16-byte lane load
  constexpr int LPK = D / EV;             // lanes per key row
  constexpr int KPI = 64 / LPK;           // key rows per load instruction of a wave
  constexpr int KPW = KPI * kDecWaves;    // key groups of the workgroup
  constexpr int BATCH = KPI * kDecUnroll;
  const int Hq = pd.n_q_heads, Hkv = pd.n_kv_heads, G = Hq / Hkv;
  const Share me = my_share<STREAM>(a);
  const int b = me.pair / Hkv, g = me.pair % Hkv;
  const int head0 = g * G + me.chunk * GC;
  const int tid = threadIdx.x, kg = tid / LPK, sub = tid % LPK;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), kgw = (tid & 63) / LPK;

  __shared__ KeyTable tab;
  __shared__ GroupSums<D, GC, KPW> sums;

  // query chunk of this lane for each head, pre-scaled so that scores are in log2 units (requested
  // first: these loads run under the table walk below)
  float qf[GC][EV];
  float slope2[GC];
  const float pos_q = BIAS ? a.new_pos[b] : 0.f;
#pragma unroll
  for (int c = 0; c < GC; ++c) {
    const T *qp = static_cast<const T *>(a.q_new) + ((int64_t)b * Hq + head0 + c) * D + sub * EV;
    Elem<T>::unpack(ld16(qp), qf[c]);
#pragma unroll
    for (int e = 0; e < EV; ++e) qf[c][e] *= a.scale * kLog2e;
    slope2[c] = BIAS ? pd.slopes[head0 + c] * kLog2e : 0.f;
  }
  const RespRows rr = resp_rows(a, b);
  if (me.chunk == 0 && blockIdx.y == 0) append_new<T, D>(pd, a, b, g, rr.write);
  build_key_table<T, D>(pd, a, b, g, rr.read, BIAS, tab);
  const RangeSearch find(tab);

  run_pieces<T, D, GC, KPW>(pd, a, me, b, head0, GC, tab.n_total, sums, [&](int key0, int key1) {
    float m[GC], l[GC], acc[GC][EV];
#pragma unroll
    for (int c = 0; c < GC; ++c) {
      m[c] = kNegBig; l[c] = 0.f;
#pragma unroll
      for (int e = 0; e < EV; ++e) acc[c][e] = 0.f;
    }
    // One batch = kDecUnroll keys per lane group, BATCH consecutive keys per wave.  Batches are software-pipelined:
    // the loads of the next batch are issued before the arithmetic of the current one (two register sets).
    struct Batch {
      u32x4 kraw[kDecUnroll], vraw[kDecUnroll];
      float pk[kDecUnroll];
    };
    auto load_batch = [&](int t0, Batch &bt) {
      const int i0 = find.uniform(t0);
      const int c0 = __builtin_amdgcn_readfirstlane(tab.cum[i0]), c1 = __builtin_amdgcn_readfirstlane(tab.cum[i0 + 1]);
      if (t0 + BATCH <= min(c1, key1)) {         // consecutive tokens of one range (nearly every batch)
        const int64_t stride = uniform64(tab.stride[i0]), off = (t0 - c0 + kgw) * stride + sub * 16;
        const char *kp = tab.k[i0] + off, *vp = tab.v[i0] + off;
#pragma unroll
        for (int u = 0; u < kDecUnroll; ++u) {
          bt.kraw[u] = ld16_kv<STREAM>(kp + u * KPI * stride);
          bt.vraw[u] = ld16_kv<STREAM>(vp + u * KPI * stride);
          bt.pk[u] = BIAS ? global_ptr<float>(tab.pos[i0])[t0 - c0 + kgw + u * KPI] : 0.f;
        }
      } else {
#pragma unroll
        for (int u = 0; u < kDecUnroll; ++u) {
          const int vk = min(t0 + kgw + u * KPI, key1 - 1);      // lanes past the end re-read the last key
          const int i = find.from(i0, vk);
          const int64_t off = int64_t(vk - tab.cum[i]) * tab.stride[i] + sub * 16;
          bt.kraw[u] = ld16_kv<STREAM>(tab.k[i] + off);
          bt.vraw[u] = ld16_kv<STREAM>(tab.v[i] + off);
          bt.pk[u] = BIAS ? global_ptr<float>(tab.pos[i])[vk - tab.cum[i]] : 0.f;
        }
      }
    };
    auto compute_batch = [&](int t0, Batch &bt) {
      if (t0 + BATCH > key1) {                   // lanes past the end: their weight is zero, but 0 * inf is not
#pragma unroll
        for (int u = 0; u < kDecUnroll; ++u)
          if (t0 + kgw + u * KPI >= key1) bt.vraw[u] = u32x4{0, 0, 0, 0};
      }
      float t[kDecUnroll][GC];
#pragma unroll
      for (int u = 0; u < kDecUnroll; ++u) {
        float kf[EV];
        Elem<T>::unpack(bt.kraw[u], kf);
#pragma unroll
        for (int c = 0; c < GC; ++c) {
          float d = 0.f;
#pragma unroll
          for (int e = 0; e < EV; ++e) d = fmaf(qf[c][e], kf[e], d);
#pragma unroll
          for (int off = LPK / 2; off >= 1; off >>= 1) d += __shfl_xor(d, off);
          // distance penalty -slope * (pos_q - pos_k), in log2 units
          t[u][c] = t0 + kgw + u * KPI < key1 ? (BIAS ? d - slope2[c] * (pos_q - bt.pk[u]) : d) : -INFINITY;
        }
      }
#pragma unroll
      for (int c = 0; c < GC; ++c) {
        float mx = t[0][c];
#pragma unroll
        for (int u = 1; u < kDecUnroll; ++u) mx = fmaxf(mx, t[u][c]);
        const float m_new = fmaxf(m[c], mx);
        const float alpha = fast_exp2(m[c] - m_new);
        m[c] = m_new;
        l[c] *= alpha;
#pragma unroll
        for (int e = 0; e < EV; ++e) acc[c][e] *= alpha;
      }
#pragma unroll
      for (int u = 0; u < kDecUnroll; ++u) {
        float vf[EV];
        Elem<T>::unpack(bt.vraw[u], vf);
#pragma unroll
        for (int c = 0; c < GC; ++c) {
          const float p = fast_exp2(t[u][c] - m[c]);
          l[c] += p;
#pragma unroll
          for (int e = 0; e < EV; ++e) acc[c][e] = fmaf(p, vf[e], acc[c][e]);
        }
      }
    };
    {
      constexpr int STEP = BATCH * kDecWaves;
      Batch b0, b1;
      int t0 = key0 + BATCH * wave;
      if (t0 < key1) load_batch(t0, b0);
      while (t0 < key1) {
        if (t0 + STEP < key1) load_batch(t0 + STEP, b1);
        compute_batch(t0, b0);
        t0 += STEP;
        if (t0 >= key1) break;
        if (t0 + STEP < key1) load_batch(t0 + STEP, b0);
        compute_batch(t0, b1);
        t0 += STEP;
      }
    }
#pragma unroll
    for (int c = 0; c < GC; ++c) {
      if (sub == 0) { sums.m[kg][c] = m[c]; sums.l[kg][c] = l[c]; }
#pragma unroll
      for (int e = 0; e < EV; ++e) sums.acc[kg][c][sub * EV + e] = acc[c][e];
    }
  });
}

// lane C of every row of 16 lanes, seen by all 16
template <int C>
__device__ __forceinline__ float row_bcast(float x) {
  return __uint_as_float(__builtin_amdgcn_mov_dpp(__float_as_uint(x), 0x150 + C, 0xf, 0xf, true));
}
// x of lane L plus (or max with) x of lane L ^ 16, L ^ 32
__device__ __forceinline__ float xrow_sum(float x) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  const float y = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(y), __float_as_uint(y), false, false);
  return __uint_as_float(s[0]) + __uint_as_float(s[1]);
}
__device__ __forceinline__ float xrow_max(float x) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  const float y = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
  const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(y), __float_as_uint(y), false, false);
  return fmaxf(__uint_as_float(s[0]), __uint_as_float(s[1]));
}
// lanes 0..31: a of lane L + a of lane L + 32; lanes 32..63: the same of b.  Likewise for even / odd rows of 16 lanes.
__device__ __forceinline__ float swap_sum32(float a, float b) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float swap_sum16(float a, float b) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
template <int I, int N, class F>
__device__ __forceinline__ void static_for(F &&f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<I + 1, N>(f);
  }
}

// bf16, several query heads per KV head.  A wave takes tiles of 16 keys:
//   S[key, head] = K[key, :] . Q[head, :]   v_mfma_f32_16x16x32_bf16, A = K rows straight from memory (lane: row
//                  lane % 16, chunks lane / 16 + 4 j), B = Q (column = head; columns past n_heads repeat a head and
//                  are not used).  Lane (g = lane / 16, h = lane % 16) then holds keys 4 g .. 4 g + 3 of head h.
//   O[head, :] += P[key, head] V[key, :]    vector unit: the lanes of row g hold V of the same keys 4 g .. 4 g + 3,
//                  16 bytes each, and take p of head h from lane h of their row (a row broadcast, no LDS).
// The vector-unit form spends a dot product and a reduction over 16 lanes per key and head; here a tile of 16 keys takes
// about 40 % of its vector instructions at four heads (64 prompts of 32/8 heads, 430 keys: 33.9 -> 25.9 us).
template <int D, int GC, bool BIAS, bool STREAM>
__global__ __launch_bounds__(kDecThreads) void decode_gqa_kernel(PlanDev pd, DecodeDev a) {
  constexpr int NJ = D / 32;                 // matrix products per tile
  constexpr int LPR = D / 8;                 // lanes per V row: 16, or 8 (then a row of 16 lanes reads two keys at once)
  constexpr int NV = LPR / 4;                // V loads per tile
  constexpr int U = 2;                       // tiles in flight per wave
  const int Hq = pd.n_q_heads, Hkv = pd.n_kv_heads, G = Hq / Hkv;
  const Share me = my_share<STREAM>(a);
  const int b = me.pair / Hkv, kvh = me.pair % Hkv;
  const int head0 = kvh * G + me.chunk * GC, n_heads = min(GC, G - me.chunk * GC);
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int g = lane >> 4, r = lane & 15, vc = lane % LPR, vhalf = LPR == 8 ? (lane >> 3) & 1 : 0;

  __shared__ KeyTable tab;
  __shared__ GroupSums<D, GC, kDecWaves> sums;

  bf16x8 qf[NJ];
  const int my_head = head0 + min(r, n_heads - 1);
#pragma unroll
  for (int j = 0; j < NJ; ++j)
    qf[j] = *reinterpret_cast<const bf16x8 *>(static_cast<const __bf16 *>(a.q_new) + ((int64_t)b * Hq + my_head) * D +
                                              (g + 4 * j) * 8);
  const float scale2 = a.scale * kLog2e;
  const float slope2 = BIAS ? pd.slopes[my_head] * kLog2e : 0.f;
  const float pos_q = BIAS ? a.new_pos[b] : 0.f;
  const RespRows rr = resp_rows(a, b);
  if (me.chunk == 0 && blockIdx.y == 0) append_new<__bf16, D>(pd, a, b, kvh, rr.write);
  build_key_table<__bf16, D>(pd, a, b, kvh, rr.read, BIAS, tab);
  const RangeSearch find(tab);

  run_pieces<__bf16, D, GC, kDecWaves>(pd, a, me, b, head0, n_heads, tab.n_total, sums, [&](int key0, int key1) {
    float m = kNegBig, l = 0.f;              // of (keys of row g, head r)
    float acc[GC][8];
#pragma unroll
    for (int h = 0; h < GC; ++h)
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[h][e] = 0.f;

    for (int t0 = key0 + 16 * U * wave; t0 < key1; t0 += 16 * U * kDecWaves) {
      bf16x8 kf[U][NJ];
      u32x4 vf[U][NV];
      float pk[U][4];
      const int i0 = find.uniform(t0);
      const int c0 = __builtin_amdgcn_readfirstlane(tab.cum[i0]), c1 = __builtin_amdgcn_readfirstlane(tab.cum[i0 + 1]);
      if (t0 + 16 * U <= min(c1, key1)) {
        // All keys of the step are consecutive tokens of one range (nearly every step).  V rows, whole in one load, are
        // read non-temporally where no other workgroup reads them; K rows are not, since four loads share a row's lines
        // (64 prompts of 32/8 heads, 590 keys: V 39.6 -> 37.5 us, both 38.4).
        const int64_t stride = uniform64(tab.stride[i0]);
        const char *kp = tab.k[i0] + (t0 - c0 + r) * stride + g * 16;
        const char *vp = tab.v[i0] + (t0 - c0 + 4 * g + vhalf) * stride + vc * 16;
#pragma unroll
        for (int u = 0; u < U; ++u) {
#pragma unroll
          for (int j = 0; j < NJ; ++j)
            kf[u][j] = *global_ptr<bf16x8>(kp + 16 * u * stride + 64 * j);
#pragma unroll
          for (int i = 0; i < NV; ++i) vf[u][i] = ld16_kv<STREAM>(vp + (16 * u + i * (LPR == 8 ? 2 : 1)) * stride);
          if (BIAS)
#pragma unroll
            for (int i = 0; i < 4; ++i) pk[u][i] = global_ptr<float>(tab.pos[i0])[t0 - c0 + 16 * u + 4 * g + i];
        }
      } else {
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int kk = min(t0 + 16 * u + r, key1 - 1), ik = find.from(i0, kk);
          const char *kp = tab.k[ik] + int64_t(kk - tab.cum[ik]) * tab.stride[ik] + g * 16;
#pragma unroll
          for (int j = 0; j < NJ; ++j) kf[u][j] = *global_ptr<bf16x8>(kp + 64 * j);
#pragma unroll
          for (int i = 0; i < NV; ++i) {
            const int vk = min(t0 + 16 * u + 4 * g + (LPR == 8 ? 2 * i + vhalf : i), key1 - 1), iv = find.from(i0, vk);
            vf[u][i] = ld16_kv<STREAM>(tab.v[iv] + int64_t(vk - tab.cum[iv]) * tab.stride[iv] + vc * 16);
          }
          if (BIAS)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const int vk = min(t0 + 16 * u + 4 * g + i, key1 - 1), iv = find.from(i0, vk);
              pk[u][i] = global_ptr<float>(tab.pos[iv])[vk - tab.cum[iv]];
            }
        }
      }
      float s[U][4], mx = -INFINITY;
#pragma unroll
      for (int u = 0; u < U; ++u) {
        f32x4 d = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < NJ; ++j) d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[u][j], qf[j], d, 0, 0, 0);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float x = BIAS ? d[i] * scale2 - slope2 * (pos_q - pk[u][i]) : d[i] * scale2;
          s[u][i] = t0 + 16 * u + 4 * g + i < key1 ? x : -INFINITY;
          mx = fmaxf(mx, s[u][i]);
        }
      }
      const float m_new = fmaxf(m, mx), alpha = fast_exp2(m - m_new);
      m = m_new;
      l *= alpha;
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          s[u][i] = fast_exp2(s[u][i] - m_new);
          l += s[u][i];
        }
      static_for<0, GC>([&](auto hc) {
        constexpr int h = decltype(hc)::value;
        const float al = row_bcast<h>(alpha);
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[h][e] *= al;
      });
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int i = 0; i < NV; ++i) {
          float v[8];
          // no V without a key: its weight is zero, but 0 * inf is not (a branch around a step's masking costs 2 %)
          const uint32_t keep = t0 + 16 * u + 4 * g + (LPR == 8 ? 2 * i + vhalf : i) < key1 ? ~0u : 0u;
          Elem<__bf16>::unpack(vf[u][i] & u32x4{keep, keep, keep, keep}, v);
          static_for<0, GC>([&](auto hc) {
            constexpr int h = decltype(hc)::value;
            float p;
            if constexpr (LPR == 16) {
              p = row_bcast<h>(s[u][i]);
            } else {
              const float p0 = row_bcast<h>(s[u][2 * i]), p1 = row_bcast<h>(s[u][2 * i + 1]);
              p = vhalf ? p1 : p0;
            }
#pragma unroll
            for (int e = 0; e < 8; ++e) acc[h][e] = fmaf(p, v[e], acc[h][e]);
          });
        }
    }
    // the four rows of lanes (and, for 64 dims, their two halves) hold different keys: one sum per wave
    const float mw = xrow_max(m), w = fast_exp2(m - mw);
    l = xrow_sum(l * w);
    if (g == 0 && r < GC) { sums.m[wave][r] = mw; sums.l[wave][r] = l; }
    static_for<0, GC>([&](auto hc) {
      constexpr int h = decltype(hc)::value;
      const float wh = row_bcast<h>(w);
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[h][e] *= wh;
    });
    // sum over the rows as a reduce-scatter: one swap and one addition take two values to one, and row g ends up with
    // the totals of values [2 GC g, 2 GC (g + 1)) of the GC x 8 (a full reduction of every value takes three times
    // the instructions, 2 us of a small launch at eight heads)
    float half[GC * 4], quarter[GC * 2];
#pragma unroll
    for (int v = 0; v < GC * 4; ++v) half[v] = swap_sum32(acc[v / 8][v % 8], acc[(v + GC * 4) / 8][v % 8]);
#pragma unroll
    for (int v = 0; v < GC * 2; ++v) {
      quarter[v] = swap_sum16(half[v], half[v + GC * 2]);
      if (LPR == 8)                                                // lane ^ 8: rotate the row by 8
        quarter[v] += __uint_as_float(__builtin_amdgcn_mov_dpp(__float_as_uint(quarter[v]), 0x128, 0xf, 0xf, true));
    }
    if (vhalf == 0) {
#pragma unroll
      for (int v = 0; v < GC * 2; ++v) {
        const int at = v + GC * 2 * g;
        sums.acc[wave][at / 8][vc * 8 + at % 8] = quarter[v];
      }
    }
  });
}

// Pieces per key list, a function of the call's arguments alone.  Measured, kernel time in us for 1 / 2 / 4 / 8 / 16
// pieces (head_dim 128; ~900 keys = 96 + 4 x 166 + response, ~160 keys = 32 + 88 + response):
//   32 heads bf16, 900 keys    1 prompt 18.3 / 13.4 / 10.8 / 9.8 / 10.9; 4: 23.5 / 18.5 / 17.3 / 16.7 / 19.6;
//                              8: 25.4 / 25.2 / 24.8 / 26.6 / 31.8; 32: 91.3 / 94.9 / 94.8 / 95.1 / 94.8
//   32/8 heads bf16, 900 keys  1 prompt 19.5 / 14.0 / 11.5 / 9.7 / 11.2; 16: 26.9 / 20.7 / 20.2 / 22.0 / 21.8;
//                              32: 31.1 / 29.0 / 31.4 / 31.4 / 31.5
//   32 heads bf16, 160 keys    1 prompt 7.7 / 8.0 / 7.6 / 7.8 / 7.8; 8: 9.4 / 11.1 / 10.6 / 14.4 / 14.4
//   32/8 heads fp32, 160 keys  1 prompt 14.6 / 12.4 / 11.1 / 9.4 / 9.4
// Hence: pieces of about 100 keys (32 where fp32 serves several heads and is bound by its vector instructions), at
// most 8 (the merge has eight pieces in flight), as many as bring two workgroups to every compute unit, and none where
// one-head workgroups fill the chip by themselves: there every piece only adds its share of the fixed cost.
constexpr int kDecMaxPieces = 8, kDecPieceKeys = 96, kDecPieceKeysF32 = 32;
static int decode_pieces(int base_wgs, int64_t rows, int64_t keys, int gc, bool bf16, int n_cu) {
  if (base_wgs > kDecPartCounters || (gc == 1 && base_wgs >= n_cu)) return 1;
  int64_t n = std::min<int64_t>(keys / (!bf16 && gc > 1 ? kDecPieceKeysF32 : kDecPieceKeys), kDecMaxPieces);
  n = std::min<int64_t>(n, (2 * n_cu + base_wgs - 1) / base_wgs);
  n = std::min<int64_t>(n, kDecPartRows / rows);
  return int(std::max<int64_t>(n, 1));
}

// How the heads of a plan are shared out: query heads per workgroup, (prompt, KV head) pairs, chunks per pair.  bf16 pads a
// group to 2, 4 or 8 columns of the matrix product (a KV head with more than 8 query heads takes several workgroups);
// fp32 takes the largest divisor of the group up to 4.
struct HeadShares { int gc, pairs, chunks; };
static HeadShares head_shares(const sp_plan *plan) {
  const int G = plan->n_q_heads / plan->n_kv_heads;
  const int gc = plan->dtype == SP_BF16 ? (G == 1 ? 1 : G == 2 ? 2 : G <= 4 ? 4 : 8) : (G % 4 == 0) ? 4 : (G % 2 == 0) ? 2 : 1;
  return {gc, plan->n_prompts * plan->n_kv_heads, (G + gc - 1) / gc};
}

void decode_scratch(const sp_plan *plan, int n_cu, size_t *part_bytes, size_t *count_bytes) {
  const HeadShares h = head_shares(plan);
  const int64_t rows = int64_t(plan->n_prompts) * plan->n_q_heads, wgs = int64_t(h.pairs) * h.chunks;
  const int most = wgs > kDecPartCounters ? 1 : decode_pieces(int(wgs), rows, INT64_MAX, h.gc, plan->dtype == SP_BF16, n_cu);
  *part_bytes = most > 1 ? (size_t(rows) * most * (plan->head_dim + 2) * 4 + 255) & ~size_t(255) : 0;
  *count_bytes = most > 1 ? (size_t(wgs) * 4 + 255) & ~size_t(255) : 0;
}

template <typename T, int D>
static hipError_t launch_decode_t(const sp_plan *plan, DecodeDev &d, const DecodeArgs &a, hipStream_t s) {
  constexpr bool kBf16 = sizeof(T) == 2;
  const HeadShares h = head_shares(plan);
  const int gc = h.gc, base = h.pairs, ny = h.chunks;
  const int64_t resp = int64_t(a.resp_len_add) + (a.resp_len ? a.resp_capacity / 2 : 0);
  const int64_t keys = plan->max_shared_keys + int64_t(a.k) * plan->max_path_keys + std::min<int64_t>(resp, a.resp_capacity);
  d.n_pieces = decode_pieces(base * ny, int64_t(plan->n_prompts) * plan->n_q_heads, keys, gc, kBf16, plan->ctx->n_cu);
  d.pieces_per_wg = d.n_pieces;
  if (d.n_pieces > 1) {
    if (const DecodeRegion *region = decode_region(plan, s)) {
      d.part = static_cast<float *>(region->part);
      d.count = region->count;
      d.pieces_per_wg = 1;
    }
  }
  d.chunks_together = ny > 1 && base % 8 == 0 && base / 8 <= 65535;
  const unsigned n_z = unsigned(d.n_pieces / d.pieces_per_wg);
  d.few_wgs = int64_t(base) * ny * n_z <= int64_t(kDecFewWgsPerCu) * plan->ctx->n_cu;
  const dim3 grid = d.chunks_together ? dim3(8u * unsigned(ny), n_z, unsigned(base) / 8) : dim3(unsigned(base), n_z, unsigned(ny));
  const dim3 block(kDecThreads);
  auto launch_as = [&](auto heads, auto bias, auto stream) {
    constexpr int GC = decltype(heads)::value;
    constexpr bool BIAS = decltype(bias)::value, STREAM = decltype(stream)::value;
    if constexpr (kBf16 && GC > 1) hipLaunchKernelGGL((decode_gqa_kernel<D, GC, BIAS, STREAM>), grid, block, 0, s, plan->dev, d);
    else if constexpr (GC <= 4) hipLaunchKernelGGL((decode_kernel<T, D, GC, BIAS, STREAM>), grid, block, 0, s, plan->dev, d);
  };
  auto launch = [&](auto heads, auto bias) {
    // bf16 has several chunks only of eight heads
    if constexpr (!kBf16 || decltype(heads)::value == 8)
      if (ny > 1) return launch_as(heads, bias, std::false_type{});
    launch_as(heads, bias, std::true_type{});
  };
  auto pick = [&](auto bias) {
    if (gc == 8) launch(std::integral_constant<int, 8>{}, bias);
    else if (gc == 4) launch(std::integral_constant<int, 4>{}, bias);
    else if (gc == 2) launch(std::integral_constant<int, 2>{}, bias);
    else launch(std::integral_constant<int, 1>{}, bias);
  };
  if (plan->has_slopes) pick(std::true_type{}); else pick(std::false_type{});
  return hipGetLastError();
}

hipError_t launch_decode(const sp_plan *plan, const DecodeArgs &a, hipStream_t s) {
  DecodeDev d{a.kept, a.k, a.Kp, a.Vp, a.kv_tok_stride, a.kv_head_stride, a.Kr, a.Vr, a.pos_resp, a.resp_capacity,
              a.resp_len, a.resp_len_add, a.new_pos, a.q_new, a.k_new, a.v_new, a.o_out, a.scale, 1, 1, nullptr, nullptr, 0, 0};
  if (plan->dtype == SP_BF16)
    return plan->head_dim == 128 ? launch_decode_t<__bf16, 128>(plan, d, a, s) : launch_decode_t<__bf16, 64>(plan, d, a, s);
  return plan->head_dim == 128 ? launch_decode_t<float, 128>(plan, d, a, s) : launch_decode_t<float, 64>(plan, d, a, s);
}

}  // namespace sp
