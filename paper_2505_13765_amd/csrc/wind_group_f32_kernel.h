// Resident groups for fp32 models: the loop of wind_group_kernel.h with fp32 weights and products.
#pragma once
#include "wind_group_kernel.h"

namespace wind {

// ---------------------------------------------------------------------------------------------
// The same loop and the same exchanges; what differs:
//   - every logit is an fp32 matrix-core product (16 x 16 x 4), so a row's argmax is taken from the exchanged (value,
//     column) words and no near-tie is decided again;
//   - weights are twice as wide: all eight waves share them (K split in eight), W_out as matrix-core operands, the
//     recurrent and the projection rows one row per lane (a matrix-vector product per emitting slot: the hidden
//     vector is read from LDS as a broadcast, nothing is summed over lanes).  One row tile per group: slots x W <= 16.
//     640 units do not quite fit (19 vector registers in scratch memory), nor 128 units with 128 labels on one CU (21);
//   - small models (GW = 1: a whole model fits one CU's registers) run one workgroup per utterance, which
//     tells itself through LDS, behind workgroup barriers: hidden vectors and projections where their readers want them, and with one
//     part of labels the rows are decided where their logits are added up.
// Bound by the chain of steps like the bf16 groups; of 640 units the products of a 16-row tile take 1.2 us (fp32 rate).
constexpr int kGroupNoLabel = 0xFFFF;   // in a word's column field; above every column
template <int NK, int CT, int GW>
struct GroupF32Cfg {
  static constexpr int H = 32 * NK, KW = H / 8;             // = Hp = Hj; a wave's part of K
  static constexpr int UPW = H / GW, NR = 4 * UPW, PPW = H / GW, NSET = (NR + PPW + 63) / 64;
  static constexpr int SL = GW == 1 ? 1 : kGroupSlots;
  static constexpr int EST = H + 4, QL = (KW + 63) / 64, NI = (4 * CT + 7) / 8;
  static_assert(PPW <= 64 || GW == 1, "the projection rows come first");
  static constexpr int PSET = (PPW + 63) / 64;               // sets of 64 rows that hold projection rows
  static constexpr size_t oE = 0;                                          // float [32][EST]
  static constexpr size_t oFred = oE + (size_t)32 * EST * 4;               // float [8][2 CT][4][80]
  static constexpr size_t oFbn = oFred + (size_t)8 * 2 * CT * 4 * 80 * 4;  // float [8][16]
  static constexpr size_t oP = oFbn + 512;                                 // float [SL][H]
  static constexpr size_t oHb = oP + (size_t)SL * H * 4;                   // float [SL][H]
  static constexpr size_t oPart = oHb + (size_t)SL * H * 4;                // float [8][SL][64 NSET]
  static constexpr size_t oRec = oPart + (size_t)8 * SL * 64 * NSET * 4;   // float [SL][NR]
  static constexpr size_t oC = oRec + (size_t)SL * NR * 4;                 // float [SL][UPW]
  static constexpr size_t oW = oC + (size_t)SL * UPW * 4;                  // float [H] blank column of W_out
  static constexpr size_t oX = (oW + (size_t)H * 4 + 15) / 16 * 16;        // GW = 1: exchange words [16][CT + 1]
  static constexpr size_t oI = oX + (GW == 1 ? (size_t)16 * (CT + 1) * 8 : 0);   // int stat[64], cnt[kNumStats], open windows [slots][2], fail, near; float bp[PPW], bo[32 CT + 1]
  static constexpr size_t oT = (oI + (64 + kNumStats + 2 * kGroupSlots + 2 + PPW + 32 * CT + 1) * 4 + 255) / 256 * 256;   // 256 bytes that group_touch writes to
  static constexpr size_t smem = oT + 256;
  static_assert(smem <= 160 * 1024, "LDS");
};

// fp32 sums of many products are kept short: what is added one after another loses half a unit in the last place of the running sum each
// time, and the per-row kernels, whose 64 lanes take a tenth of a sum each and add in a tree, set the measure.  Blocks of 8
// products, added in pairs, then over the wave's part of K, the eight waves' parts as a tree, the bias last.  Logits of
// 640 units against 64 bits: one chain per wave 2.6e-7 rms, the per-row kernels 1.2e-7, the blocks 1.3e-7
// (batch of 8, 600 frames: 1.44 -> 1.55 ms)
template <class F>
__device__ __forceinline__ float group_sum8(const F &f) {
  return ((f(0) + f(1)) + (f(2) + f(3))) + ((f(4) + f(5)) + (f(6) + f(7)));
}
// Sum of w[n] h[FROM + n] for n = 0 .. 7, h[m] from lane m of the lane's row of 16 (DPP row_newbcast).  One block of
// assembly: the compiler keeps the broadcasts as moves of their own, which doubles the instructions; the no-op in
// front keeps the required distance from whatever wrote h.
template <int FROM>
__device__ __forceinline__ float group_row_products(float h, const float *w) {
  static_assert(FROM == 0 || FROM == 8, "half a row of lanes");
  float a = 0.f;
#define WIND_FMAC(n, lane) "v_fmac_f32_dpp %0, %1, %" #n " row_newbcast:" #lane " row_mask:0xf bank_mask:0xf"
  if constexpr (FROM == 0)
    asm("s_nop 1\n\t" WIND_FMAC(2, 0) "\n\t" WIND_FMAC(3, 1) "\n\t" WIND_FMAC(4, 2) "\n\t" WIND_FMAC(5, 3) "\n\t" WIND_FMAC(6, 4) "\n\t"
        WIND_FMAC(7, 5) "\n\t" WIND_FMAC(8, 6) "\n\t" WIND_FMAC(9, 7)
        : "+v"(a)
        : "v"(h), "v"(w[0]), "v"(w[1]), "v"(w[2]), "v"(w[3]), "v"(w[4]), "v"(w[5]), "v"(w[6]), "v"(w[7]));
  else
    asm("s_nop 1\n\t" WIND_FMAC(2, 8) "\n\t" WIND_FMAC(3, 9) "\n\t" WIND_FMAC(4, 10) "\n\t" WIND_FMAC(5, 11) "\n\t" WIND_FMAC(6, 12) "\n\t"
        WIND_FMAC(7, 13) "\n\t" WIND_FMAC(8, 14) "\n\t" WIND_FMAC(9, 15)
        : "+v"(a)
        : "v"(h), "v"(w[0]), "v"(w[1]), "v"(w[2]), "v"(w[3]), "v"(w[4]), "v"(w[5]), "v"(w[6]), "v"(w[7]));
#undef WIND_FMAC
  return a;
}

template <int NK, int CT, int GW, int MODE>   // MODE: kGroupMany, ..
__global__ __launch_bounds__(512) void wind_group_f32_kernel(ModelDev m, CallDev c, GroupDev gd) {
  using Cfg = GroupF32Cfg<NK, CT, GW>;
  constexpr int H = Cfg::H, KW = Cfg::KW, NR = Cfg::NR, PPW = Cfg::PPW, QL = Cfg::QL, NSET = Cfg::NSET;
  constexpr bool SOLO = GW == 1, ONE = SOLO || MODE != kGroupMany, LIM = MODE == kGroupLimited;
  constexpr int SL = ONE ? 1 : Cfg::SL;
  constexpr bool kDirect = SOLO && CT == 1;   // one part of columns, and it is here
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  const int grp = SOLO ? (int)blockIdx.x : (int)blockIdx.x % kGroups, g = SOLO ? 0 : (int)blockIdx.x / kGroups;
  if (grp >= gd.NG) return;
  if (blockIdx.x == 0 && threadIdx.x == 0) c.stats[kStatLoop] = (unsigned long long)wall_clock64();
  float *ecache = reinterpret_cast<float *>(smem + Cfg::oE), *fred = reinterpret_cast<float *>(smem + Cfg::oFred);
  float *fbn = reinterpret_cast<float *>(smem + Cfg::oFbn), *pfull = reinterpret_cast<float *>(smem + Cfg::oP);
  float *hbuf = reinterpret_cast<float *>(smem + Cfg::oHb), *partl = reinterpret_cast<float *>(smem + Cfg::oPart);
  float *recs = reinterpret_cast<float *>(smem + Cfg::oRec), *cst = reinterpret_cast<float *>(smem + Cfg::oC);
  float *wbl = reinterpret_cast<float *>(smem + Cfg::oW);
  int *stat = reinterpret_cast<int *>(smem + Cfg::oI), *counts = stat + 64, *fail = counts + kNumStats + 2 * kGroupSlots, *near_w = fail + 1;
  float *bpl = reinterpret_cast<float *>(near_w + 1), *bol = bpl + PPW;   // this workgroup's rows of b_pred, columns of b_out and blank's

  int lane = threadIdx.x & 63, tid = threadIdx.x, l15 = lane & 15, l4 = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int W = c.W, V = m.V, NS = gd.NS, W2 = 2 * W, R = NS * W, nparts = c.nparts_tiny, kstride = nparts + 1;
  unsigned *abort_word = SOLO ? nullptr : gd.bar + grp * kGroupBarInts;
  unsigned long long *xs = reinterpret_cast<unsigned long long *>(smem + Cfg::oX);
  unsigned long long *hx = gd.h_x + (size_t)grp * kGroupSlots * H, *px = gd.p_x + (size_t)grp * kGroupSlots * H;   // not SOLO
  unsigned long long *kbase = SOLO ? xs : gd.keys + (size_t)grp * 2 * kGroupRows * kstride;
  const int unit0 = g * Cfg::UPW, prow0 = g * PPW;
  const int n_order = *gd.n_order;
  GroupLane sl = group_first_slots<ONE>(c, gd, grp, lane, n_order);
  GroupOpen open{0, 0};

  // ---- weights into registers
  float wo[2 * CT][NK], wv[NSET][KW];
#pragma unroll
  for (int t = 0; t < 2 * CT; ++t) {
    const int col = min(((t >> 1) * GW + g) * 32 + 16 * (t & 1) + l15, m.Vpad - 1);
    const float *src = reinterpret_cast<const float *>(m.w_out) + (size_t)col * H + wave * KW + l4 * NK;
#pragma unroll
    for (int i = 0; i < NK; ++i) wo[t][i] = src[i];
  }
#pragma unroll
  for (int t = 0; t < NSET; ++t) {
    const int r = t * 64 + lane;
    const float *src = (r < PPW ? reinterpret_cast<const float *>(m.w_pred) + (size_t)(prow0 + r) * H
                                : reinterpret_cast<const float *>(m.w_cat[0]) + (size_t)(unit0 * 4 + min(r - PPW, NR - 1)) * H) + wave * KW;
#pragma unroll
    for (int i = 0; i < KW; ++i) wv[t][i] = src[i];
  }
  auto load_frames = [&]() { group_load_frames<H, Cfg::EST>(c, gd, sl, ecache, 0, lane, wave, 8); };

  // ---- state after the start token
  for (int i = tid; i < NS * H; i += 512) pfull[i] = m.start_p[i % H];
  for (int i = tid; i < H; i += 512) wbl[i] = m.w_blank[i];
  for (int i = tid; i < NS * NR; i += 512) recs[i] = m.start_rec[unit0 * 4 + i % NR];
  for (int i = tid; i < NS * Cfg::UPW; i += 512) cst[i] = m.start_c[unit0 + i % Cfg::UPW];
  for (int i = tid; i < kNumStats + 2 * kGroupSlots; i += 512) counts[i] = 0;
  for (int i = tid; i < PPW; i += 512) bpl[i] = m.b_pred[prow0 + i];
  for (int i = tid; i <= 32 * CT; i += 512) {
    const int part = (i >> 5) * GW + g, col = i < 32 * CT ? part * 32 + (i & 31) : V;
    bol[i] = i == 32 * CT || (part < nparts && col < V) ? m.b_out[col] : kKeyNone;   // what is added to kKeyNone vanishes in it
  }
  load_frames();
  if (tid == 0) { *fail = 0; *near_w = 1; }
  // ---- where the workgroups sit: XCD numbers, exchanged with device-wide stores
  if (!SOLO && wave == 0) {
    unsigned xcc;
    asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(xcc));
    xcc = (xcc & 15u) + 1u;
    unsigned *bw = abort_word + 64;
    if (lane == 0) __hip_atomic_store(bw + g * 32, xcc, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    unsigned v = xcc;
    const bool got = group_poll(abort_word, gd.start_limit, [&]() {
      if (lane < GW) v = __hip_atomic_load(bw + lane * 32, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      return v != 0u;
    });
    const bool same = __all(v == xcc);
    if (lane == 0) {
      *near_w = (same ? 1 : 0) | (group_keys_suffice(nparts, GW, 1) ? 0 : 2);
      if (!got) *fail = 1;
      if (g == 0) abort_word[1] = same ? 2u : 1u;
    }
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  group_barrier();
  const int flags = __builtin_amdgcn_readfirstlane(*near_w);
  const bool near = flags & 1, publishes = flags & 2;
  auto put = [&](unsigned long long *p, unsigned lo, unsigned hi) {
    if constexpr (SOLO) *p = (unsigned long long)lo | ((unsigned long long)hi << 32);
    else group_st(p, lo, hi, near);
  };
  auto get = [&](const unsigned long long *p) {
    if constexpr (SOLO) return *p;
    else return group_ld(p);
  };
  auto wait = [&](const auto &ask) {   // SOLO: the words are behind a workgroup barrier
    if constexpr (SOLO) { ask(); return true; }
    else return group_poll(abort_word, gd.spin_limit, ask);
  };

  const unsigned touch_lds = (unsigned)(unsigned long long)(__attribute__((address_space(3))) unsigned char *)(smem + Cfg::oT);
  const unsigned winv = 65536u / (unsigned)W + 1u;   // x / W for x < 64
  auto div_w = [&](int x) { return (int)(((unsigned)x * winv) >> 16); };
  int pend = 0, pend_slot[kGroupSlots] = {0, 0, 0, 0};

  for (int it = 0;; ++it) {
    asm volatile("" : "+v"(lane), "+v"(tid));   // see group_loop
    l15 = lane & 15;
    l4 = lane >> 4;
    const int nwin = group_window<LIM>(c, gd, sl, open);   // lanes of empty slots: 0
    if (!__any(nwin > 0)) break;
    const unsigned stamp = (unsigned)it + 1u, stamp16 = stamp & 0xFFFFu;
    unsigned long long *kp = SOLO ? kbase : kbase + (size_t)group_key_buffer(it) * kGroupRows * kstride;
    if constexpr (!SOLO) {   // the keys that this iteration's replace have been read by everybody
      if (publishes && wave == 6 && group_keys_need(it) > 0 &&
          !group_poll(abort_word, gd.spin_limit, [&]() { return group_decided<GW>(abort_word + 32, lane, group_keys_need(it)); }) && lane == 0) *fail = 1;
    }
    {
      // ---- window rows as matrix-core operands: lane (row l15, K group l4), NK consecutive units of this wave's part of K
      f32x4 acc[2 * CT];
#pragma unroll
      for (int t = 0; t < 2 * CT; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
      const int gq = div_w(l15), ga = gq < NS ? gq : 0, gj = gq < NS ? l15 - ga * W : 0;
      int rr = (ONE ? __builtin_amdgcn_readfirstlane(sl.rpos) : __shfl(sl.rpos, ga, kWave)) + gj;
      if (rr >= W2) rr -= W2;
      const float *er = ecache + (ga * W2 + rr) * Cfg::EST + wave * KW + l4 * NK;
      const float *pr = pfull + ga * H + wave * KW + l4 * NK, *br = wbl + wave * KW + l4 * NK;
      float dot = 0.f;
      constexpr int VEC = NK % 4 == 0 ? 4 : 2;
#pragma unroll
      for (int i = 0; i < NK; i += VEC) {
        float ev[VEC], pv[VEC], bv[VEC];
        if constexpr (VEC == 4) {
          const float4 e4 = *reinterpret_cast<const float4 *>(er + i), p4 = *reinterpret_cast<const float4 *>(pr + i), b4 = *reinterpret_cast<const float4 *>(br + i);
          ev[0] = e4.x; ev[1] = e4.y; ev[2] = e4.z; ev[3] = e4.w;
          pv[0] = p4.x; pv[1] = p4.y; pv[2] = p4.z; pv[3] = p4.w;
          bv[0] = b4.x; bv[1] = b4.y; bv[2] = b4.z; bv[3] = b4.w;
        } else {
          const float2 e2 = *reinterpret_cast<const float2 *>(er + i), p2 = *reinterpret_cast<const float2 *>(pr + i), b2 = *reinterpret_cast<const float2 *>(br + i);
          ev[0] = e2.x; ev[1] = e2.y; pv[0] = p2.x; pv[1] = p2.y; bv[0] = b2.x; bv[1] = b2.y;
        }
        constexpr int NB = CT == 1 ? 2 : 1, STEPS = VEC / NB;   // blocks of 8 products (VEC 2: 4); 16 where the registers hold four parts of W_out
        f32x4 blk[NB][2 * CT];                                  // a matrix-core product adds four of a row's
        float d = 0.f;
#pragma unroll
        for (int q = 0; q < VEC; ++q) {
          const float z = fmaxf(ev[q] + pv[q], 0.f);
          d = fmaf(z, bv[q], d);
#pragma unroll
          for (int t = 0; t < 2 * CT; ++t)
            blk[q / STEPS][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(z, wo[t][i + q], q % STEPS ? blk[q / STEPS][t] : f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
        }
        dot += d;
#pragma unroll
        for (int t = 0; t < 2 * CT; ++t) acc[t] += NB == 2 ? blk[0][t] + blk[NB - 1][t] : blk[0][t];
        __builtin_amdgcn_sched_barrier(0);   // a block's LDS operands at a time: registers
      }
      dot = quarter_sum(dot);
#pragma unroll
      for (int t = 0; t < 2 * CT; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) fred[((wave * 2 * CT + t) * 4 + r) * 80 + lane] = acc[t][r];
      if (lane < 16) fbn[wave * 16 + lane] = dot;
    }
    group_barrier();   // B1
    // ---- best label of every (row, part): item (row quad q4, part): lane = (row 4 q4 + l4, columns l15 and l15 + 16)
#pragma unroll
    for (int k = 0; k < Cfg::NI; ++k) {
      const int item = wave + 8 * k;
      if (item >= 4 * CT) continue;
      const int q4 = item & 3, ct = item >> 2, part = ct * GW + g;
      float v[2];
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        v[t] = group_sum8([&](int w) { return fred[((w * 2 * CT + 2 * ct + t) * 4 + l4) * 80 + 16 * q4 + l15]; }) + bol[ct * 32 + 16 * t + l15];
      }
      // a NaN (from infinite frames) is no label's: the maxima pass over it, and a part of nothing else has column kGroupNoLabel
      const float b = fmaxf(v[0], v[1]), bm = row16_max_f32(b);
      const int at = part * 32 + l15 + (v[0] == b ? 0 : 16);   // ties: the lower column
      const int col = kGroupNoLabel - row16_max_i32(b == bm ? kGroupNoLabel - at : 0);
      const int row = 4 * q4 + l4;
      if constexpr (kDirect) {   // all labels are in this part: the row is decided here
        const float blank = group_sum8([&](int w) { return fbn[w * 16 + row]; }) + bol[32 * CT];
        // blank has the highest id: it wins only if strictly larger, and where no label has a logit
        const int label = row >= __builtin_amdgcn_readfirstlane(nwin) || col >= V || !(bm >= kKeyNone) || blank > bm ? V : col;
        if (l15 == 0) stat[row] = label;
        if (label < V && l15 < min((NR * 4 + 127) / 128 + 1, 16))   // see group_loop
          group_touch(m.emb_gates + (unsigned)label * (4u * H) + (unsigned)min(l15 * 32, NR - 1), touch_lds);
      } else if (part < nparts && l15 == 0 && row < R) put(kp + row * kstride + part, __float_as_uint(bm), (unsigned)(col & 0xFFFF) | (stamp16 << 16));
    }
    if (!kDirect && wave == 4 && g == 0 && lane < R) {   // R <= 16
      const float d2 = group_sum8([&](int w) { return fbn[w * 16 + lane]; }) + bol[32 * CT];
      put(kp + lane * kstride + nparts, __float_as_uint(d2), stamp16 << 16);
    }
    if (wave >= 4)   // the recurrent sums of the last step
      for (int i = tid - 256; i < pend * NR; i += 256) {
        const int e = i / NR, row = i - e * NR;
        const float v = group_sum8([&](int w) { return partl[(w * SL + e) * 64 * NSET + PPW + row]; });
        const int s = e == 0 ? pend_slot[0] : e == 1 ? pend_slot[1] : e == 2 ? pend_slot[2] : pend_slot[3];
        recs[s * NR + row] = v;
      }
    pend = 0;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the last iteration's frames have landed
    // ---- exchange 1: four rows per wave, 16 lanes per row
    if constexpr (SOLO && !kDirect) group_barrier();
    if (!kDirect && 4 * wave < R) {
      const int row = 4 * wave + l4, a = div_w(row);
      const bool valid = ONE ? row < __builtin_amdgcn_readfirstlane(nwin) : row - a * W < __shfl(nwin, a, kWave);   // one slot: no row past its window
      unsigned long long kA = 0ull, kB = 0ull, kC = 0ull;
      const bool got = wait([&]() {
        if (!valid) return true;
        const unsigned long long *kr = kp + row * kstride;
        if (l15 < nparts) kA = get(kr + l15);
        if (l15 + 16 < nparts) kB = get(kr + l15 + 16);
        kC = get(kr + nparts);
        return (l15 >= nparts || (unsigned)(kA >> 48) == stamp16) && (l15 + 16 >= nparts || (unsigned)(kB >> 48) == stamp16) &&
               (unsigned)(kC >> 48) == stamp16;
      });
      if (!got && lane == 0) *fail = 1;
      float b = kKeyNone;
      int col = kGroupNoLabel;
      if (valid && l15 < nparts) {
        b = __uint_as_float((unsigned)kA);
        col = (int)(kA >> 32) & 0xFFFF;
      }
      if (valid && l15 + 16 < nparts && (__uint_as_float((unsigned)kB) > b || b != b)) {   // ties: the lower column
        b = __uint_as_float((unsigned)kB);
        col = (int)(kB >> 32) & 0xFFFF;
      }
      const float bm = row16_max_f32(b);
      col = kGroupNoLabel - row16_max_i32(b == bm ? kGroupNoLabel - col : 0);
      // blank has the highest id: it wins only if strictly larger, and where no label has a logit
      const int label = !valid || col >= V || __uint_as_float((unsigned)kC) > bm ? V : col;
      if (l15 == 0) stat[row] = label;
      if (label < V && l15 < min((NR * 4 + 127) / 128 + 1, 16))   // see group_loop
        group_touch(m.emb_gates + (unsigned)label * (4u * H) + (unsigned)(unit0 * 4 + min(l15 * 32, NR - 1)), touch_lds);
    }
    group_barrier();   // B2
    if (*fail) return;
    if constexpr (!SOLO) {
      if (publishes && wave == 6 && lane == 0) group_publish(abort_word + 32 + g, stamp, near);   // this workgroup's reads of the keys are done
    }
    const int lab = lane < R ? stat[lane] : V;
    const unsigned long long m_nb = __ballot(lab != V);
    int tok;
    bool emits, fresh_slot;
    group_outcome<LIM, ONE>(c, gd, sl, open, grp, lane, n_order, nwin, V, m_nb, 0ull, lab, wave == 7 && g == 0, counts, tok, emits, fresh_slot);
    const unsigned long long em = __ballot(emits), rf = __ballot(fresh_slot);
    if (em) {
      const int n_em = ONE ? 1 : __popcll(em);
      int es[kGroupSlots] = {0, 0, 0, 0}, et[kGroupSlots] = {0, 0, 0, 0};
      {
        unsigned long long todo = em;
#pragma unroll
        for (int e = 0; e < SL; ++e)
          if (todo) {
            es[e] = __builtin_amdgcn_readfirstlane(__ffsll((long long)todo) - 1);
            et[e] = __builtin_amdgcn_readlane(tok, es[e]);
            todo &= todo - 1;
          }
      }
      // ---- LSTM step: thread (emitting slot, gate row of this workgroup's units)
      // A thread has one at most.  As a loop over the threads' items it left by its last lane into a block where, with 640 units, the compiler
      // put the constant 1 into a register before it took the lanes back: a wait that gave up then stored whatever was there
      // as its failure
      static_assert(SL * NR <= 512 && SL * PPW <= 512, "a thread each");
      if (tid < n_em * NR) {
        const int le = tid / NR, li = tid - le * NR;
        const int s = le == 0 ? es[0] : le == 1 ? es[1] : le == 2 ? es[2] : es[3], tk = le == 0 ? et[0] : le == 1 ? et[1] : le == 2 ? et[2] : et[3];
        const float pre = recs[s * NR + li] + m.emb_gates[(unsigned)tk * (4u * H) + (unsigned)(unit0 * 4 + li)];   // fits 32 bits: checked by the host
        const float act = (li & 3) == 2 ? tanhf(pre) : 1.f / (1.f + expf(-pre));
        const float ig = dpp_f32<0x00>(act), fg = dpp_f32<0x55>(act), gg = dpp_f32<0xAA>(act), og = dpp_f32<0xFF>(act);   // the unit's four gates
        if ((li & 3) == 0) {
          const int u = li >> 2;
          const float cn = fg * cst[s * Cfg::UPW + u] + ig * gg;
          cst[s * Cfg::UPW + u] = cn;
          if constexpr (SOLO) hbuf[u] = og * tanhf(cn);
          else put(hx + s * H + unit0 + u, __float_as_uint(og * tanhf(cn)), stamp);
        }
      }
      // ---- exchange 2 / 3: this wave's part of the emitting slots' vectors, into its part of `to`
      auto fetch = [&](const unsigned long long *from, float *to, bool by_slot) {
        unsigned long long u[SL][QL];
        const bool got = wait([&]() {
          bool fresh = true;
#pragma unroll
          for (int e = 0; e < SL; ++e)
            if (e < n_em) {
#pragma unroll
              for (int q = 0; q < QL; ++q) u[e][q] = get(from + es[e] * H + wave * KW + min(lane + 64 * q, KW - 1));
            }
#pragma unroll
          for (int e = 0; e < SL; ++e)
            if (e < n_em) {
#pragma unroll
              for (int q = 0; q < QL; ++q) fresh = fresh && (unsigned)(u[e][q] >> 32) == stamp;
            }
          return fresh;
        });
        if (!got && lane == 0) *fail = 1;
#pragma unroll
        for (int e = 0; e < SL; ++e)
          if (e < n_em) {
#pragma unroll
            for (int q = 0; q < QL; ++q)
              if (lane + 64 * q < KW) to[(by_slot ? es[e] : e) * H + wave * KW + lane + 64 * q] = __uint_as_float((unsigned)u[e][q]);
          }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // read back by this wave only
      };
      // rows of set `t` times the e-th new hidden vector, over this wave's part of K.  The vector sits in registers, 16 values
      // to a register in every row of 16 lanes, and each product takes its value from its row's lane n (as an LDS
      // broadcast per value the reads bound this: 0.75 us for 80 values)
      float hv[(KW + 15) / 16];
      auto take_vector = [&](int e) {
#pragma unroll
        for (int i = 0; i < (KW + 15) / 16; ++i) hv[i] = hbuf[e * H + wave * KW + min(16 * i + l15, KW - 1)];
      };
      auto row_sums = [&](int t, int e) {
        static_assert(KW == 8 || KW % 16 == 0, "whole blocks");
        float a = group_row_products<0>(hv[0], wv[t]);
        if constexpr (KW > 8) a += group_row_products<8>(hv[0], wv[t] + 8);
#pragma unroll
        for (int i = 16; i < KW; i += 16) a += group_row_products<0>(hv[i / 16], wv[t] + i) + group_row_products<8>(hv[i / 16], wv[t] + i + 8);
        partl[(wave * SL + e) * 64 * NSET + t * 64 + lane] = a;
      };
      if constexpr (SOLO) group_barrier();
      else fetch(hx, hbuf, false);
      for (int e = 0; e < n_em; ++e) {
        take_vector(e);
#pragma unroll
        for (int t = 0; t < Cfg::PSET; ++t) row_sums(t, e);
      }
      group_barrier();   // B3: partial sums of the projection rows
      if (tid < n_em * PPW) {
        const int e = tid / PPW, row = tid - e * PPW;
        const float v = group_sum8([&](int w) { return partl[(w * SL + e) * 64 * NSET + row]; });
        const int s = e == 0 ? es[0] : e == 1 ? es[1] : e == 2 ? es[2] : es[3];
        if constexpr (SOLO) pfull[row] = v + bpl[row];
        else put(px + s * H + prow0 + row, __float_as_uint(v + bpl[row]), stamp);
      }
      // ---- while the projections travel: the recurrent sums of the next step (added behind the next barrier)
      for (int e = 0; e < n_em; ++e) {
        take_vector(e);
#pragma unroll
        for (int t = Cfg::PSET; t < NSET; ++t) row_sums(t, e);
      }
      pend = n_em;
#pragma unroll
      for (int e = 0; e < SL; ++e) pend_slot[e] = es[e];
      if constexpr (SOLO) group_barrier();
      else fetch(px, pfull, true);
    }
    load_frames();
    if (rf) {   // slots that took a new utterance: the state after the start token, their first frames
      unsigned long long todo = rf;
      while (todo) {
        const int a = __builtin_amdgcn_readfirstlane(__ffsll((long long)todo) - 1);
        todo &= todo - 1;
        for (int i = tid; i < H; i += 512) pfull[a * H + i] = m.start_p[i];
        for (int i = tid; i < NR; i += 512) recs[a * NR + i] = m.start_rec[unit0 * 4 + i];
        for (int i = tid; i < Cfg::UPW; i += 512) cst[a * Cfg::UPW + i] = m.start_c[unit0 + i];
      }
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      group_barrier();
    }
  }
  if (g == 0 && wave == 7) group_add_counters(c, counts, lane);
}

// ---------------------------------------------------------------------------------------------
// e = W_enc enc + b_enc of fp32 models: 64 x 64 tiles, fp32 matrix-core products (32 x 32 x 2), one 32 x 32 block per wave,
// both operands through LDS in stages of 32 inputs, the next stage's loads in flight during a stage's
// products.  D a multiple of 4 (other models: enc_proj_f32_kernel).  A row tile is 64 frames of one utterance.
__global__ __launch_bounds__(256) void enc_proj_f32_tile_kernel(ModelDev m, CallDev c, int tiles_per_utt, GroupDev gd, int init_blocks) {
  constexpr int BK = 32, ST = BK + 4;
  __shared__ __attribute__((aligned(16))) float as[64 * ST], bs[64 * ST];
  if ((int)blockIdx.x < init_blocks) {
    if (blockIdx.y == 0) group_init(m, c, gd, (int)blockIdx.x, init_blocks, reinterpret_cast<int *>(as));
    return;
  }
  const int tile = (int)blockIdx.x - init_blocks, b = tile / tiles_per_utt, t0 = (tile % tiles_per_utt) * 64, n0 = blockIdx.y * 64, D = m.D;
  const int len = utt_len(c, b);
  if (t0 >= len) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, wm = wave >> 1, wn = wave & 1;
  // thread: rows tid / 8 and tid / 8 + 32 of both tiles, inputs 4 (tid & 7) ..
  const int lr = tid >> 3, lk = (tid & 7) * 4;
  const float *ap[2], *bp[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    ap[h] = c.enc + ((size_t)b * c.T + min(t0 + lr + 32 * h, len - 1)) * D + lk;
    bp[h] = reinterpret_cast<const float *>(m.w_enc) + (size_t)(n0 + lr + 32 * h) * D + lk;   // rows up to a multiple of 256 exist
  }
  float4 av[2], bv[2];
  auto fetch = [&](int k0) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      av[h] = bv[h] = make_float4(0.f, 0.f, 0.f, 0.f);
      if (k0 + lk < D) {
        av[h] = *reinterpret_cast<const float4 *>(ap[h] + k0);
        bv[h] = *reinterpret_cast<const float4 *>(bp[h] + k0);
      }
    }
  };
  // sums as short as above: blocks of 8 inputs (part), in pairs over a stage of 32, over four stages (run), over those.  D = 1024, rms
  // against 64 bits: one chain 5.7e-7, the per-row kernel 1.0e-7, the blocks 1.0e-7 (8 x 600 frames: 63 -> 85 us)
  f32x16 acc, run, zero;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = run[r] = zero[r] = 0.f;
  fetch(0);
  for (int k0 = 0; k0 < D; k0 += BK) {
    __syncthreads();
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      *reinterpret_cast<float4 *>(&as[(lr + 32 * h) * ST + lk]) = av[h];
      *reinterpret_cast<float4 *>(&bs[(lr + 32 * h) * ST + lk]) = bv[h];
    }
    __syncthreads();
    if (k0 + BK < D) fetch(k0 + BK);
    // lane (row or column lane & 31, half lane >> 5) takes inputs 16 half + 0 .. 15 of the stage, two per product step
    const float *ar = &as[(wm * 32 + (lane & 31)) * ST + (lane >> 5) * 16], *br = &bs[(wn * 32 + (lane & 31)) * ST + (lane >> 5) * 16];
    f32x16 part[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float4 a4 = *reinterpret_cast<const float4 *>(ar + 4 * i), b4 = *reinterpret_cast<const float4 *>(br + 4 * i);
      part[i] = __builtin_amdgcn_mfma_f32_32x32x2f32(a4.x, b4.x, zero, 0, 0, 0);
      part[i] = __builtin_amdgcn_mfma_f32_32x32x2f32(a4.y, b4.y, part[i], 0, 0, 0);
      part[i] = __builtin_amdgcn_mfma_f32_32x32x2f32(a4.z, b4.z, part[i], 0, 0, 0);
      part[i] = __builtin_amdgcn_mfma_f32_32x32x2f32(a4.w, b4.w, part[i], 0, 0, 0);
    }
    run += (part[0] + part[1]) + (part[2] + part[3]);
    if (((k0 / BK) & 3) == 3) {
      acc += run;
      run = zero;
    }
  }
  acc += run;
  const int col = n0 + wn * 32 + (lane & 31);
  if (col >= m.Hj) return;
  const float bias = m.b_enc[col];
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int t = t0 + wm * 32 + acc_row(0, r, lane);
    if (t < len) c.e[((size_t)b * c.T + t) * m.Hj + col] = acc[r] + bias;
  }
}

}  // namespace wind
