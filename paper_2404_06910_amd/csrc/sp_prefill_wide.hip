// a1 (bf16 storage, 128 dims): ForkJoin prefill attention where many rows see the same long key list, a fork behind a chain of
// kept documents above all (iterative superposition, Sec. 4.1.2).  The mask and the products are those of the other bf16
// kernel (Sec. 3.2, 3.2.1); what differs is who loads and how much a load serves.
//
// There a workgroup is two waves of 32 rows, and each wave issues eight DMA instructions per block of 32 keys between its
// products.  A compute unit takes some 124 lines of misses at a time, so those instructions wait for each other, and with
// them the wave that is to compute: a fifth of its time goes by in the issue, as much again in the wait for what was issued
// one stage ago.  Here a workgroup is a whole compute unit: 8 waves of 32 rows compute and 4 waves do nothing but load, three
// stages of 64 keys ahead, so that a wait in the issue costs no product, and a K/V row that is fetched serves 256 rows
// instead of 64.  Three waves per SIMD leave 168 registers to each, which the 64-key block fits (8 products of 32x32x16 for
// each half, one softmax) as long as no address is kept from stage to stage.
//
// The rows of a tile may come from several row groups when these fork behind the same segment: the short rests of 16 sibling
// paths would each stream the whole chain by themselves.  A tile's keys are one virtual sequence [ancestors ; own run of each
// group], each part beginning at a multiple of 32, so that a block of 32 keys is the ancestors' or one group's.
//
// Waves do not meet in barriers.  A loader wave counts a slot of the ring filled when its part has landed, a computing wave
// counts it read when its last LDS read of it has returned; each waits for the count that it needs.  Loaders wait for
// readers of earlier stages, all of which they have announced before they wait; readers wait for loaders; all walk the same
// sequence of stages, so every wait ends.
//
// Measured, 8 prompts of 16 documents of 128 + 24 tokens behind 576 tokens in five ranges, 32 heads of 128 dims (208 GFLOP):
// 363 us with the other kernel, 301 here.  Before the parts came together: with loads issued by the 8 computing waves and a
// barrier per stage 370 us; 4 computing waves of their own loads, two workgroups per compute unit 358; these with two loader
// waves 372 (a ring of two stages is all that fits); loaders, barriers and Q rows straight into registers 311; counters for
// the barriers 310; Q rows through the ring 305; O rows straight from the registers, without LDS, 301.  Without its loads and
// stores the kernel takes 264 us, without its arithmetic 165.
#include "sp_device.h"
#include "sp_internal.h"
#include "sp_lds_dma.h"

namespace sp {

namespace {

constexpr int D = 128, ROWB = 2 * D, NJ = D / 16, NC = D / 32;
constexpr int NW = kWideWaves;
constexpr int BK = kWideStageKeys;                 // keys of a stage
constexpr int SLOTS = 4;                           // stages in LDS: a stage is 64 K rows and 64 V rows, or 128 Q rows
constexpr int HALFB = BK * ROWB, STAGEB = 2 * HALFB;
constexpr int NP = 4;                              // loader waves
constexpr int LROWS = 2 * BK / NP, NDMA = LROWS / 4;   // rows of a stage that a loader wave fetches, 4 per DMA instruction
constexpr int NQ = NW / NP;                         // stages of Q rows
constexpr int kBatch = 24;                         // items staged in LDS at a time
constexpr int kTileVec = sizeof(WideTile) / 16;
static_assert(sizeof(WideTile) % 16 == 0 && alignof(WideTile) == 16, "tiles are moved in pieces of 16 bytes");
static_assert(NDMA == 8, "the waits count eight DMA instructions per stage");

}  // namespace

template <int HPW, bool BIAS>
__global__ __launch_bounds__(64 * (NW + NP), 3) void prefill_wide_kernel(PlanDev pd, const __bf16 *__restrict__ Q,
                                                                  const __bf16 *__restrict__ K,
                                                                  const __bf16 *__restrict__ V, __bf16 *__restrict__ O,
                                                                  uint32_t q_ts, uint32_t q_hs, uint32_t kv_ts,
                                                                  uint32_t kv_hs, float scale) {
  __shared__ __attribute__((aligned(1024))) unsigned char ring[SLOTS * STAGEB];
  __shared__ __attribute__((aligned(256))) float Ps[BIAS ? SLOTS : 1][NP][64];  // positions of a stage's keys or of Q rows
  __shared__ WideTile s_tiles[kBatch];
  __shared__ int s_heads[kBatch];
  // how often a loader wave has filled a slot, how often a computing wave has read it
  __shared__ int s_filled[SLOTS], s_read[SLOTS];

  const int wg_slot = (blockIdx.x % 8) * (pd.n_wg / 8) + blockIdx.x / 8;
  const int x0 = pd.wg_begin[wg_slot], n_mine = pd.wg_begin[wg_slot + 1] - x0;
  if (n_mine <= 0) return;

  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const float scale2 = scale * kLog2e;
  const uint32_t ring_base = (uint32_t)(size_t)(lds_byte *)ring;
  const uint32_t ps_base = (uint32_t)(size_t)(lds_byte *)&Ps[0][0][0];
  // The lane's number, taken anew wherever addresses are made of it: kept from stage to stage they cost some forty registers
  // and spill, and a reload waits for every DMA in flight.
  auto lane_now = [&]() {
    int l = tid & 63;
    asm volatile("" : "+v"(l));
    return l;
  };

  // The first half of the loader waves fills the K rows of a stage, the others the V rows.
  const int loader = wave - NW;
  const bool dma_is_v = loader >= NP / 2;
  const int rbase = LROWS * (loader % (NP / 2));
  const uint32_t dstep = dma_is_v ? 0 : 64;                          // chunk offset of instruction m: dch ^ (m % 4) * dstep
  const char *const KVb = reinterpret_cast<const char *>(dma_is_v ? V : K);

  auto issue = [&](int li, int kv_head, int st, int slot) {
    const int lane = lane_now(), drow = lane >> 4;
    const uint32_t dch = (uint32_t)((lane & 15) ^ (dma_is_v ? 4 * drow : drow)) * 16;
    const uint32_t kv_row_off = (uint32_t)drow * kv_ts * 2;
    const uint32_t lds = ring_base + slot * STAGEB + loader * (LROWS * ROWB);
    const int vk0 = st * BK;
    const WideRange *const rg = s_tiles[li].range;
    const int4 e = *reinterpret_cast<const int4 *>(&rg[lane % kWideRanges]);
    const int r = __builtin_ctz(uint32_t(__ballot(vk0 < e.y)) | 1u << (kWideRanges - 1));
    const int delta = __builtin_amdgcn_readlane(e.x, r), end = __builtin_amdgcn_readlane(e.y, r),
              last = __builtin_amdgcn_readlane(e.z, r);
    const uint64_t hoff = (uint64_t)(uint32_t)kv_head * kv_hs * 2;
    auto token = [&](int vk) -> int {
      int d = delta, en = end, la = last;
      for (int q = r + 1; q < kWideRanges && __any(vk >= en); ++q) {
        const int4 x = *reinterpret_cast<const int4 *>(&rg[q]);
        if (vk >= en) { d = x.x; en = x.y; la = x.z; }
      }
      return min(d + vk, la);
    };
    if (vk0 + BK <= end && delta + vk0 + BK - 1 <= last) {
      const uint64_t o0 = (uint64_t)(uint32_t)(delta + vk0 + rbase) * kv_ts * 2 + hoff;
#pragma unroll
      for (int m = 0; m < NDMA; ++m)
        dma16s(KVb + (o0 + (uint64_t)(4 * m) * kv_ts * 2), kv_row_off + (dch ^ (m % 4 * dstep)), lds + m * (4 * ROWB));
      if (BIAS && loader == 0) dma4(pd.tok_pos + (delta + vk0 + lane), ps_base + slot * (NP * 256));
    } else {
#pragma unroll
      for (int m = 0; m < NDMA; ++m) {
        const int tok = token(vk0 + rbase + 4 * m + drow);
        dma16(KVb + ((uint64_t)(uint32_t)tok * kv_ts * 2 + hoff + (dch ^ (m % 4 * dstep))), lds + m * (4 * ROWB));
      }
      if (BIAS && loader == 0) dma4(pd.tok_pos + token(vk0 + lane), ps_base + slot * (NP * 256));
    }
  };

  // One lane adds; a counter at or past `want` is waited for.
  auto count = [&](int *c) {
    if ((tid & 63) == 0) __hip_atomic_fetch_add(c, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  };
  auto reached = [&](int *c, int want) {
    return __builtin_amdgcn_readfirstlane(__hip_atomic_load(c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) >= want;
  };
  if (tid < SLOTS) s_filled[tid] = s_read[tid] = 0;
  int seq = 0;                                             // stages since the kernel began

  bf16x8 qf[NJ];
  f32x16 o[NC];
  float m_run = kNegBig, l_run = 0.f, slope2 = 0.f, pos_q = 0.f;

  // rows of block i of an item
  struct Rows { int tok, n_rows, first, base; };
  auto rows_of = [&](int li, int i) -> Rows {
    const int4 a = *reinterpret_cast<const int4 *>(&s_tiles[li].block[i]);
    return {__builtin_amdgcn_readfirstlane(a.x), __builtin_amdgcn_readfirstlane(a.y), __builtin_amdgcn_readfirstlane(a.z),
            __builtin_amdgcn_readfirstlane(a.w)};
  };
  // Q rows of a computing wave, as K rows are: loader i fetches those of wave NP * part + i
  auto issue_q = [&](int li, int part, int slot) {
    const int lane = lane_now(), drow = lane >> 4, w = NP * part + loader;
    const Rows rw = rows_of(li, w / HPW);
    const int head = (__builtin_amdgcn_readfirstlane(s_heads[li]) & 0xffff) + w % HPW, top = max(rw.n_rows - 1, 0);
    const uint32_t lds = ring_base + slot * STAGEB + loader * (32 * ROWB);
    const uint64_t o0 = ((uint64_t)(uint32_t)rw.tok * q_ts + (uint64_t)(uint32_t)head * q_hs) * 2;
    const uint32_t ch = (uint32_t)((lane & 15) ^ drow) * 16;
#pragma unroll
    for (int m = 0; m < 8; ++m)                            // rows past the block repeat its last row
      dma16s(reinterpret_cast<const char *>(Q) + o0, (uint32_t)min(4 * m + drow, top) * q_ts * 2 + (ch ^ (m % 4 * 64)),
             lds + m * (4 * ROWB));
    if (BIAS) dma4(pd.tok_pos + rw.tok + min(lane, top), ps_base + (slot * NP + loader) * 256);
  };

  for (int batch = 0; batch < n_mine; batch += kBatch) {
    const int n_it = min(kBatch, n_mine - batch);
    __syncthreads();
    for (int i = tid; i < n_it * kTileVec; i += 64 * (NW + NP)) {
      const int li = i / kTileVec, part = i % kTileVec;
      reinterpret_cast<int4 *>(&s_tiles[li])[part] =
          reinterpret_cast<const int4 *>(pd.wide_tiles + pd.wide_items[x0 + batch + li].tile)[part];
    }
    if (tid < n_it) s_heads[tid] = pd.wide_items[x0 + batch + tid].heads;
    __syncthreads();

    auto kv_of = [&](int li) { return int(uint32_t(__builtin_amdgcn_readfirstlane(s_heads[li])) >> 16); };
    auto stages_of = [&](int li) { return (__builtin_amdgcn_readfirstlane(s_tiles[li].n_keys) + BK - 1) / BK; };
    if (wave >= NW) {
      __builtin_amdgcn_s_setprio(3);
      int li = 0, st = -NQ, ns = stages_of(0), kv = kv_of(0);
      int told = seq;                                      // stages that the computing waves know of
#pragma unroll 1
      while (li < n_it) {
        const int slot = seq % SLOTS, want = NW * (seq / SLOTS);
        if (!reached(&s_read[slot], want)) {
          // the ring is full: everything under way lands meanwhile
          asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
          for (; told < seq; ++told) count(&s_filled[told % SLOTS]);
          while (!reached(&s_read[slot], want)) __builtin_amdgcn_s_sleep(1);
        }
        asm volatile("" ::: "memory");
        if (st < 0) issue_q(li, st + NQ, slot);
        else issue(li, kv, st, slot);
        ++seq;
        if (seq - told > 2) {
          asm volatile("s_waitcnt vmcnt(16)" ::: "memory");   // all but the last two stages
          count(&s_filled[told++ % SLOTS]);
        }
        if (++st == ns) {
          st = -NQ;
          if (++li < n_it) { ns = stages_of(li); kv = kv_of(li); }
        }
      }
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      for (; told < seq; ++told) count(&s_filled[told % SLOTS]);
      continue;
    }

    auto wait_filled = [&]() {
      while (!reached(&s_filled[seq % SLOTS], NP * (seq / SLOTS + 1))) __builtin_amdgcn_s_sleep(1);
      asm volatile("" ::: "memory");
    };
    auto release = [&]() {
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      count(&s_read[seq % SLOTS]);
      ++seq;
    };
#pragma unroll 1
    for (int it = 0; it < n_it; ++it) {
      const Rows w = rows_of(it, wave / HPW);
      const int head = (__builtin_amdgcn_readfirstlane(s_heads[it]) & 0xffff) + wave % HPW;
      const int ns = stages_of(it), anc = __builtin_amdgcn_readfirstlane(s_tiles[it].anc),
                anc_end = __builtin_amdgcn_readfirstlane(s_tiles[it].anc_end);
      const int w_last = w.first + w.n_rows - 1;           // no rows: below the first key
      // Stages of other waves' rows are waited for too: a slot that is counted as read before all have read what it held
      // could be filled under a reader.
      auto pass = [&]() { wait_filled(); release(); };
      for (int part = 0; part < wave / NP; ++part) pass();
      wait_filled();
      {
        const int lane = lane_now(), l32 = lane & 31, half = lane >> 5;
        const uint32_t qb = (seq % SLOTS) * STAGEB + ((wave % NP) * 32 + l32) * ROWB + ((half ^ l32) & 15) * 16;
#pragma unroll
        for (int j = 0; j < NJ; ++j) qf[j] = *reinterpret_cast<const bf16x8 *>(ring + (qb ^ (32 * j)));
        if (BIAS) {
          pos_q = Ps[seq % SLOTS][wave % NP][l32];
          slope2 = sload_f32(pd.slopes + head) * kLog2e;
        }
      }
      release();
      for (int part = wave / NP + 1; part < NQ; ++part) pass();
#pragma unroll
      for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int i = 0; i < 16; ++i) o[c][i] = 0.f;
      m_run = kNegBig;
      l_run = 0.f;

#pragma unroll 1
      for (int st = 0; st < ns; ++st) {
        wait_filled();
        const int slot = seq % SLOTS;
        const int lane = lane_now(), l32 = lane & 31, half = lane >> 5, tr_row = (lane & 15) >> 2;
        const int my_limit = w.first + min(l32, max(w.n_rows - 1, 0));
        // K row l32, chunk 2j + half: kb ^ 32j; V rows 4 half + tr_row on, dims 32c on: vb ^ 64c
        const uint32_t kb = slot * STAGEB + l32 * ROWB + ((half ^ l32) & 15) * 16;
        const uint32_t vb = slot * STAGEB + HALFB + (4 * half + tr_row) * ROWB + (lane & 1) * 8 +
                            (4 * tr_row + 2 * ((lane >> 4) & 1) + ((lane & 3) >> 1)) * 16;
        const int vk0 = st * BK;
        const bool last = st + 1 == ns;
        auto sees = [&](int b) { return w.n_rows > 0 && (b < anc_end || (b + 31 >= w.base && b <= w_last)); };
        const bool lo = sees(vk0), hi = sees(vk0 + 32);
        if (lo || hi) {
          // Both halves of the stage in one softmax.  (Where the wave sees one half, leaving the other out of the scores too
          // takes 21-30 spilled registers: 306 us where this takes 301.)
          f32x16 s[2];
#pragma unroll
          for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int i = 0; i < 16; ++i) s[b][i] = 0.f;
          __builtin_amdgcn_s_setprio(1);
#pragma unroll
          for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int b = 0; b < 2; ++b)
              s[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                  *reinterpret_cast<const bf16x8 *>(ring + (32 * b) * ROWB + (kb ^ (32 * j))), qf[j], s[b], 0, 0, 0);
          __builtin_amdgcn_s_setprio(0);
#pragma unroll
          for (int b = 0; b < 2; ++b) {
            const int b0 = vk0 + 32 * b;
            if (BIAS) {
#pragma unroll
              for (int q = 0; q < 4; ++q) {
                const f32x4 kp = *reinterpret_cast<const f32x4 *>(&Ps[slot][0][32 * b + 8 * q + 4 * half]);
#pragma unroll
                for (int i = 0; i < 4; ++i) s[b][4 * q + i] = fmaf(s[b][4 * q + i], scale2, slope2 * (kp[i] - pos_q));
              }
            }
            // last visible key: of the ancestors, or this lane's row; no key of a run that lies before the wave's own
            const bool shared = b0 < anc_end, other = !shared && b0 < w.base;
            if (b0 + 31 > (shared ? anc - 1 : w.first) || other) {
              const int lim = (shared ? anc - 1 : other ? -1 : my_limit) - b0 - 4 * half;
#pragma unroll
              for (int i = 0; i < 16; ++i)
                if (8 * (i / 4) + (i % 4) > lim || other) s[b][i] = -INFINITY;
            }
          }
          float mx = fmaxf(s[0][0], s[0][1]);
#pragma unroll
          for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int i = b ? 0 : 2; i < 16; ++i) mx = fmaxf(mx, s[b][i]);
          if (!BIAS) mx *= scale2;                         // scale2 > 0: max commutes with the scaling
          mx = xhalf_max(mx);
          // as in the other kernel, the reference may lag behind the maximum by 8
          if (__any(mx > m_run + 8.f)) {
            const float m_new = fmaxf(m_run, mx);
            const float alpha = fast_exp2(m_run - m_new);
            m_run = m_new;
            l_run *= alpha;
#pragma unroll
            for (int c = 0; c < NC; ++c)
#pragma unroll
              for (int i = 0; i < 16; ++i) o[c][i] *= alpha;
          }
          bf16x8 pb[4];
#pragma unroll
          for (int b = 0; b < 2; ++b) {
            float ls = 0.f;
#pragma unroll
            for (int i = 0; i < 16; ++i) {
              const float p = BIAS ? fast_exp2(s[b][i] - m_run) : fast_exp2(fmaf(s[b][i], scale2, -m_run));
              ls += p;
              pb[2 * b + i / 8][i % 8] = static_cast<__bf16>(p);
            }
            l_run += ls;
          }
          // V of a half that the wave does not see is not touched: it may be another path's, and zero times an infinity is NaN
          __builtin_amdgcn_s_setprio(1);
#pragma unroll
          for (int b = 0; b < 2; ++b)
            if (b ? hi : lo) {
#pragma unroll
              for (int mm = 2 * b; mm < 2 * b + 2; ++mm)
#pragma unroll
                for (int c = 0; c < NC; ++c) {
                  const unsigned char *vp = ring + 16 * mm * ROWB + (vb ^ (64 * c));
                  const bf16x4 v0 = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4 *)vp);
                  const bf16x4 v1 = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4 *)(vp + 8 * ROWB));
                  o[c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_shufflevector(v0, v1, 0, 1, 2, 3, 4, 5, 6, 7), pb[mm],
                                                                 o[c], 0, 0, 0);
                }
            }
          __builtin_amdgcn_s_setprio(0);
        }
        release();
        if (last) {
          if (w.n_rows > 0) {
            const float inv = 1.f / xhalf_sum(l_run);
            char *const ob = reinterpret_cast<char *>(O) +
                             ((uint64_t)(uint32_t)w.tok * q_ts + (uint64_t)(uint32_t)head * q_hs) * 2;
            // Lane L holds dims 8q + 4 (L / 32) + (0..3) of row L % 32.  Two groups of eight dims change halves with lane L ^ 32,
            // and each lane stores eight dims in a row.  Rows past the block hold what its last row holds, and go there.
            const uint32_t off = (uint32_t)min(l32, w.n_rows - 1) * q_ts * 2 + 16 * half;
#pragma unroll
            for (int c = 0; c < NC; ++c)
#pragma unroll
              for (int q = 0; q < 4; q += 2) {
                u32x4 v;
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                  bf16x2 lo, hi;
#pragma unroll
                  for (int i = 0; i < 2; ++i) {
                    lo[i] = static_cast<__bf16>(o[c][4 * q + 2 * e + i] * inv);
                    hi[i] = static_cast<__bf16>(o[c][4 * q + 4 + 2 * e + i] * inv);
                  }
                  const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, lo), __builtin_bit_cast(uint32_t, hi),
                                                                  false, false);
                  v[e] = r[0];
                  v[2 + e] = r[1];
                }
                st16(ob + (off + 64 * c + 16 * q), v);
              }
          }
        }
      }
    }
  }
}

template <int HPW>
static hipError_t launch_hpw(const sp_plan *plan, const PrefillArgs &a, hipStream_t s) {
  const dim3 grid(unsigned(plan->dev.n_wg));
  const __bf16 *Q = static_cast<const __bf16 *>(a.Q), *K = static_cast<const __bf16 *>(a.K),
               *V = static_cast<const __bf16 *>(a.V);
  __bf16 *O = static_cast<__bf16 *>(a.O);
  const uint32_t qts = uint32_t(a.q_tok_stride), qhs = uint32_t(a.q_head_stride), kts = uint32_t(a.kv_tok_stride),
                 khs = uint32_t(a.kv_head_stride);
  if (plan->has_slopes)
    hipLaunchKernelGGL((prefill_wide_kernel<HPW, true>), grid, dim3(64 * (NW + NP)), 0, s, plan->dev, Q, K, V, O, qts, qhs, kts, khs,
                       a.scale);
  else
    hipLaunchKernelGGL((prefill_wide_kernel<HPW, false>), grid, dim3(64 * (NW + NP)), 0, s, plan->dev, Q, K, V, O, qts, qhs, kts, khs,
                       a.scale);
  return hipGetLastError();
}

hipError_t launch_prefill_wide(const sp_plan *plan, const PrefillArgs &a, hipStream_t s) {
  switch (plan->heads_per_wg) {
    case 2: return launch_hpw<2>(plan, a, s);
    default: return launch_hpw<1>(plan, a, s);
  }
}

}  // namespace sp
