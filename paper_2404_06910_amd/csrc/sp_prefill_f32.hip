// a1 (fp32 storage): ForkJoin prefill attention over the prompt DAG (Sec. 3.2, 3.2.1; App. B.3), the precision path
// (tolerance 1e-4), on the fp32 matrix instruction: inputs, products, sums and probabilities stay in 32 bits.
//
// A work item of the plan is up to tile_rows (16, 32 or 64) consecutive rows of one row group for HPW query heads that share
// a KV head.  It is done by one-wave workgroups; a wave owns 16 of its rows of one head and walks the rows' keys (ancestor ranges
// root to leaf, then the own run up to its last row) 16 at a time.  Per step, with v_mfma_f32_16x16x4_f32:
//   S^T[key, row] = K[key, :] . Q[row, :]        A = K, B = Q (registers for the whole item)
//   O^T[d, row]  += V^T[d, key] . P^T[key, row]  A = V, B = P as the first product leaves it
// Lane L holds row L % 16 throughout: accumulator register r of a 16x16 tile is its row 4 * (L / 16) + r, which is also
// the k-slot that lane feeds in the second product when slot L / 16 of step r is bound to key 4 * (L / 16) + r.  So the
// probabilities never move.  The k-slots of the first product and the rows of O^T are bound so that every lane reads and
// writes 16-byte vectors: dims 16i + 4 * (L / 16) + e of K and Q, dims 64h + 4 * (L % 16) + e of V.
//
// What bounds it: the matrix pipe (a loop of these products alone sustains 120 TFLOP/s on this part).  K and V fragments
// are loaded straight from memory into registers, V under the first product, the next K under the second, and no wave
// waits for another.  16 rows per wave and not 32: a masked half of a diagonal tile and an unfilled last tile cost half as
// much, and the waves are short enough for the last of them to end together.  Sums are kept in short chains that are then
// added up: one chain of D products (and one of all keys for O) has 1.75 times the error of one wave per row in vector
// arithmetic, the short ones have 0.80 to 0.99 of it (against 64 bits, four shapes).
// Measured, one prompt of 20 documents of 64-220 tokens, 32 heads of 128 dims (9.9 GFLOP): 712 us with one wave per row in
// vector arithmetic, 161 us now.  In a profiled run, where it takes 176: 194 us with the waves of an item in one workgroup
// (it keeps its place until its longest wave ends), 209 us with K and V staged through LDS for the four waves of an item.
// Without the early K loads, at three waves per SIMD: 183 us where this one took 164.
#include <algorithm>

#include "sp_device.h"
#include "sp_internal.h"

namespace sp {

namespace {

// value of a row's four lanes (L, L ^ 16, L ^ 32, L ^ 48) combined
__device__ __forceinline__ float quad_max(float x) {
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
__device__ __forceinline__ float quad_sum(float x) {
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = __uint_as_float(a[0]) + __uint_as_float(a[1]);
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

}  // namespace

template <int D, int HPW, bool BIAS>
__global__ __launch_bounds__(64, 2) void prefill_f32_kernel(PlanDev pd, const float *__restrict__ Q,
                                                                  const float *__restrict__ K,
                                                                  const float *__restrict__ V, float *__restrict__ O,
                                                                  int64_t q_ts, int64_t q_hs, int64_t kv_ts,
                                                                  int64_t kv_hs, float scale, int log2_waves,
                                                                  int first_round) {
  constexpr int NI = D / 16;             // 16-byte vectors of a K or Q row per lane; 16-wide blocks of O^T
  constexpr int NH = D / 64;
  // A block is one wave.  Blocks are dealt round-robin over the 8 XCDs and started in order: the waves of an item follow
  // each other on one XCD, and an XCD works on a window of consecutive items of its own range of the list (slot
  // x * (n_wg / 8) + i holds the items of XCD x that are i-th in its order, then the (i + n_wg / 8)-th, and so on).
  const int xcd = blockIdx.x % 8, nth = blockIdx.x / 8, wave = nth & ((1 << log2_waves) - 1), per_xcd = pd.n_wg / 8;
  const int slot = xcd * per_xcd + (nth >> log2_waves) % per_xcd;
  const int item = pd.wg_begin[slot] + first_round + (nth >> log2_waves) / per_xcd;
  if (item >= pd.wg_begin[slot + 1]) return;
  const WorkItem w = pd.items[item];

  const int lane = threadIdx.x;
  const int l16 = lane & 15, quad = lane >> 4;
  const int head = (w.head0 & 0xffff) + wave % HPW;
  const int r0 = 16 * (wave / HPW);                          // first tile row of this wave
  if (r0 >= w.n_rows) return;
  const int rows = min(16, w.n_rows - r0);
  const int row = r0 + min(l16, rows - 1);                   // lanes past the tile repeat its last row
  const int row_tok = w.tok_start + w.row0 + row;
  const int my_limit = w.anc_keys + w.row0 + row;            // last virtual key that this lane's row sees
  const int first_limit = w.anc_keys + w.row0 + r0, last_limit = first_limit + rows - 1;
  const int64_t kv_head = uint32_t(w.head0) >> 16;
  const float *Kh = K + kv_head * kv_hs + 4 * quad;
  const float *Vg = V + kv_head * kv_hs, *Vh = Vg + 4 * l16;

  // The key range that holds virtual key `base`: [base, base + len) are the tokens from tok on.  Range n_ranges is the
  // own run.  base, len and tok are the same for all lanes.
  int rng = -1, base = 0, len = 0, tok = 0;
  // Range r, or the own run behind the last one (from virtual key b on).  The table is read in either case (a group without
  // ranges reads the entry at its place in it, or the padding behind the table): a choice between two places to read from
  // becomes a choice of addresses, with a flat load and a spilled register in every step that ends a range.
  auto range = [&](int r, int b) -> KeyRange {
    const KeyRange kr = pd.ranges[w.range_off + max(min(r, w.n_ranges - 1), 0)];
    const bool own = r >= w.n_ranges;
    return {own ? w.tok_start : kr.tok_start, own ? 0x7fffffff - b : kr.len};
  };
  auto seek = [&](int vk) {
    while (vk >= base + len) {
      base += len;
      const KeyRange kr = range(++rng, base);
      tok = kr.tok_start;
      len = kr.len;
    }
  };
  // token of virtual key vk >= base; keys behind the last visible one (masked) repeat that one
  auto token_of = [&](int vk) -> int {
    int r = rng, b = base, n = len, t = tok;
    vk = min(vk, last_limit);
    while (vk >= b + n) {
      b += n;
      const KeyRange kr = range(++r, b);
      t = kr.tok_start;
      n = kr.len;
    }
    return t + (vk - b);
  };

  float q[4 * NI];
  {
    const float *qp = Q + int64_t(row_tok) * q_ts + int64_t(head) * q_hs + 4 * quad;
    const float scale2 = scale * kLog2e;
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const f32x4 v = *reinterpret_cast<const f32x4 *>(qp + 16 * i);
#pragma unroll
      for (int e = 0; e < 4; ++e) q[4 * i + e] = v[e] * scale2;
    }
  }
  const float slope2 = BIAS ? pd.slopes[head] * kLog2e : 0.f;
  const float pos_q = BIAS ? pd.tok_pos[row_tok] : 0.f;

  f32x4 o[NI];                       // o[4h + c][r]: dim 64h + 16 quad + 4r + c of this lane's row
#pragma unroll
  for (int c = 0; c < NI; ++c)
#pragma unroll
    for (int r = 0; r < 4; ++r) o[c][r] = 0.f;
  float m = kNegBig, l = 0.f;
  f32x4 kf[NI], vf[NI][4];           // vf[h][r]: dims 64h + 4 l16 + (0..3) of key 4 quad + r
  int vtok[4];                       // tokens of keys 4 quad + r of the step whose K is in kf

  auto load_k = [&](int vk0) {
    seek(vk0);
    int ktok;
    if (vk0 + 15 < base + len && vk0 + 15 <= last_limit) {   // 16 consecutive tokens
      const int t0 = tok + (vk0 - base);
      ktok = t0 + l16;
#pragma unroll
      for (int r = 0; r < 4; ++r) vtok[r] = t0 + 4 * quad + r;
    } else {
      ktok = token_of(vk0 + l16);
#pragma unroll
      for (int r = 0; r < 4; ++r) vtok[r] = __shfl(ktok, 4 * quad + r);
    }
    const float *kp = Kh + int64_t(ktok) * kv_ts;
#pragma unroll
    for (int i = 0; i < NI; ++i) kf[i] = *reinterpret_cast<const f32x4 *>(kp + 16 * i);
  };

  load_k(0);
  for (int vk0 = 0; vk0 <= last_limit; vk0 += 16) {
    float kpos[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float *vp = Vh + int64_t(vtok[r]) * kv_ts;
#pragma unroll
      for (int h = 0; h < NH; ++h) vf[h][r] = *reinterpret_cast<const f32x4 *>(vp + 64 * h);
      if (BIAS) kpos[r] = pd.tok_pos[vtok[r]];
    }
    const int step_tok[4] = {vtok[0], vtok[1], vtok[2], vtok[3]};

    // one short chain of products per 16 dims, added up pairwise: the rounding of a single chain of D products is
    // several times larger
    f32x4 s[NI];
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      f32x4 a = {0.f, 0.f, 0.f, 0.f}, b = a;
      a = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[i][0], q[4 * i], a, 0, 0, 0);
      b = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[i][1], q[4 * i + 1], b, 0, 0, 0);
      a = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[i][2], q[4 * i + 2], a, 0, 0, 0);
      b = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[i][3], q[4 * i + 3], b, 0, 0, 0);
      s[i] = a + b;
    }
#pragma unroll
    for (int n = NI / 2; n >= 1; n /= 2)
#pragma unroll
      for (int i = 0; i < n; ++i) s[i] += s[i + n];
    if (vk0 + 16 <= last_limit) load_k(vk0 + 16);

    const bool diag = vk0 + 15 > first_limit;                // some row sees only part of these keys
    float t[4], p[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      t[r] = s[0][r];
      if (BIAS) t[r] -= slope2 * (pos_q - kpos[r]);
      if (diag && vk0 + 4 * quad + r > my_limit) t[r] = -INFINITY;
    }
    const float mx = quad_max(fmaxf(fmaxf(t[0], t[1]), fmaxf(t[2], t[3])));
    // The reference is the maximum itself, as soon as it grows: one that may lag behind it saves 0.5 % of the time and lets
    // sums overflow early, one that is set above it costs precision (1.67e-7 of the norm against 1.06e-7) and denormals.
    if (__any(mx > m)) {
      const float m_new = fmaxf(m, mx), alpha = fast_exp2(m - m_new);
      m = m_new;
      l *= alpha;
#pragma unroll
      for (int c = 0; c < NI; ++c)
#pragma unroll
        for (int r = 0; r < 4; ++r) o[c][r] *= alpha;
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) p[r] = fast_exp2(t[r] - m);
    l += (p[0] + p[1]) + (p[2] + p[3]);

    bool plain = true;
    if (diag) {
      // The product below multiplies the V row of a key that a row does not see by zero, which leaves no trace only
      // while that V row is finite.
      float z = 0.f;
#pragma unroll
      for (int h = 0; h < NH; ++h)
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
          for (int c = 0; c < 4; ++c) z = fmaf(vf[h][r][c], 0.f, z);
      plain = !__any(z != 0.f);
    }
    if (plain) {
      // a sum of its own per 16 keys, for the same reason
#pragma unroll
      for (int h = 0; h < NH; ++h) {
        f32x4 a[4], b[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) a[c] = b[c] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int r = 0; r < 4; r += 2)
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            a[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[h][r][c], p[r], a[c], 0, 0, 0);
            b[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[h][r + 1][c], p[r + 1], b[c], 0, 0, 0);
          }
#pragma unroll
        for (int c = 0; c < 4; ++c) o[4 * h + c] += a[c] + b[c];
      }
    } else {
      for (int kk = 0; kk < 16; ++kk) {
        const int src = 16 * (kk >> 2);
        const float p0 = __shfl(p[0], src + l16), p1 = __shfl(p[1], src + l16), p2 = __shfl(p[2], src + l16),
                    p3 = __shfl(p[3], src + l16);
        const int t0 = __shfl(step_tok[0], src), t1 = __shfl(step_tok[1], src), t2 = __shfl(step_tok[2], src),
                  t3 = __shfl(step_tok[3], src);
        const int e = kk & 3;
        const float pk = e == 0 ? p0 : e == 1 ? p1 : e == 2 ? p2 : p3;
        const int tk = e == 0 ? t0 : e == 1 ? t1 : e == 2 ? t2 : t3;
        if (vk0 + kk > my_limit) continue;
        const float *vp = Vg + int64_t(tk) * kv_ts + 16 * quad;
#pragma unroll
        for (int c = 0; c < NI; ++c)
#pragma unroll
          for (int r = 0; r < 4; ++r) o[c][r] = fmaf(pk, vp[64 * (c / 4) + 4 * r + c % 4], o[c][r]);
      }
    }
  }

  const float inv = 1.f / quad_sum(l);
  if (l16 >= rows) return;
  float *op = O + int64_t(row_tok) * q_ts + int64_t(head) * q_hs + 16 * quad;
#pragma unroll
  for (int h = 0; h < NH; ++h)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      f32x4 v;
#pragma unroll
      for (int c = 0; c < 4; ++c) v[c] = o[4 * h + c][r] * inv;
      *reinterpret_cast<f32x4 *>(op + 64 * h + 4 * r) = v;
    }
}

template <int D, int HPW>
static hipError_t launch_hpw(const sp_plan *plan, const PrefillArgs &a, hipStream_t s) {
  const float *Q = static_cast<const float *>(a.Q), *K = static_cast<const float *>(a.K),
              *V = static_cast<const float *>(a.V);
  float *O = static_cast<float *>(a.O);
  // one wave per 16 tile rows and head; rounds of one item per slot, in as many launches as 2^32 threads each allow
  const int waves = plan->tile_rows / 16 * HPW, log2_waves = __builtin_ctz(unsigned(waves));
  const int most = int((int64_t(1) << 32) / (int64_t(plan->n_wg) * waves * 64)) - 1;
  for (int first = 0; first < plan->max_slice; first += most) {
    const dim3 grid(unsigned(plan->n_wg) * unsigned(std::min(plan->max_slice - first, most)) * unsigned(waves));
    if (plan->has_slopes)
      hipLaunchKernelGGL((prefill_f32_kernel<D, HPW, true>), grid, dim3(64), 0, s, plan->dev, Q, K, V, O, a.q_tok_stride,
                         a.q_head_stride, a.kv_tok_stride, a.kv_head_stride, a.scale, log2_waves, first);
    else
      hipLaunchKernelGGL((prefill_f32_kernel<D, HPW, false>), grid, dim3(64), 0, s, plan->dev, Q, K, V, O, a.q_tok_stride,
                         a.q_head_stride, a.kv_tok_stride, a.kv_head_stride, a.scale, log2_waves, first);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;                                         // no round: every segment is cached
}

template <int D>
static hipError_t launch_d(const sp_plan *plan, const PrefillArgs &a, hipStream_t s) {
  switch (plan->heads_per_wg) {
    case 4: return launch_hpw<D, 4>(plan, a, s);
    case 2: return launch_hpw<D, 2>(plan, a, s);
    default: return launch_hpw<D, 1>(plan, a, s);
  }
}

hipError_t launch_prefill_f32(const sp_plan *plan, const PrefillArgs &a, hipStream_t s) {
  return plan->head_dim == 128 ? launch_d<128>(plan, a, s) : launch_d<64>(plan, a, s);
}

}  // namespace sp
