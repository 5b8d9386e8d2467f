// Beam search on resident workgroups: the passes of a search without a launch and without a wait for the stream, and one scoring
// step as a single launch, or as four that wait for nobody.
#pragma once
#include "wind_beam.h"
#include "wind_group_kernel.h"

namespace wind {

// ---------------------------------------------------------------------------------------------
// A pass of the search (prediction-network step of the new label sequences, joiner rows, soft-max, K best pairs) is a chain of
// steps that are far too short for launches of their own: five launches, each with its start, its first loads and its drain, and
// a wait for the stream took 45 us for 20 MFLOP.  Here 32 workgroups on one XCD (one per CU) stay on the chip with the model's
// weights in registers as matrix-core operands, and exchange through that XCD's L2 as the resident groups of the decoder do: every
// 8-byte word carries the number of the command it belongs to, a reader asks until all it needs are of its own.
// 640 units, 1024 labels, K = 4, windows of 16: a command takes 14.7 us as the host sees it: network step 3.8 (two exchanges),
// projections 1.3, logits 2.4, soft-max rows 2.1, merge 2.2, the bus and the pass-on 2.9; a search of 250 frames 51.1 -> 24.1 ms (18.7 to 20 with the host's part as it is now).
//
// Commands come from the host, one per pass, through pinned memory, results go back the same way, both as such words: a pass is one
// trip over the bus each way (about 2 us), four exchanges in the L2 and the steps between them.
// Workgroup 0 alone watches for commands and passes them on to the others, so that all of them agree on what comes next; when
// none has come for `idle_ticks` it sends everybody away, and the host launches the kernel again with the command that it
// has by then.  A command is sent only when the results of the one before are back, and passed on only when every
// workgroup is done with that one: no word is overwritten before its readers have it.  Every other wait is bounded by spin_limit
// (the first one, for all workgroups to be on the chip, by start_limit); a wave that gives up sets the abort word, all leave, and
// the host runs the rest of the search with launches.
//
// The state slots (h, c, p) carry no numbers and are read through each CU's own vector cache: a slot is written once in a launch, by all workgroups,
// and no line of it is read before that (the host hands out slots that rise and never come back, and every index that is clamped, for
// lanes or sequences beyond the last, is clamped to one that the command names).  Whoever uses a slot again has to read it past that cache.
//
// Workgroup g: columns 32 g .. 32 g + 31 of W_out (the blank of 1024-label models: workgroup 31 as well), 4 KS LSTM units, 4 KS rows
// of W_pred.  K is split in four over the waves of a half; the halves (waves 0-3 and 4-7) share the row tiles of the logits and the recurrent
// rows, and the first has the projection's.
constexpr int kBeamResWgs = 32;
constexpr int kBeamResHyps = 8;       // hypotheses of a pass, and new label sequences
constexpr int kBeamResRows = 128;     // joiner rows of a command
constexpr int kBeamResFrames = 16;    // frames of a window
constexpr int kBeamPrefixRows = 16;      // rows of a prefix-step command
constexpr int kBeamLgStride = 1040;   // words of a row of logits: 65 tiles of 16 columns
constexpr int kBeamRowWords = 2 + 2 * kBeamResHyps;   // what a row leaves for the merge: log-sum-exp, log P(blank), K candidates
constexpr int kBeamCmdWords = 64, kBeamResultWords = kBeamResHyps * kBeamResHyps;
constexpr int kBeamCodeNone = 0x7FFF;   // in a result word: no such pair
enum { kBeamCmdQuit = 0, kBeamCmdScore = 1, kBeamCmdComplete = 2 };
enum { kBeamExitIdle = 1, kBeamExitFailed = 2, kBeamExitAsked = 3 };
// Places in a command.  A hypothesis' word: its slot, and above that 1 + which of the new sequences it is (0: none of them)
enum { kBeamAtHead = 0, kBeamAtFrame = 1, kBeamAtK = 2, kBeamAtParent = 3, kBeamAtChild = 11, kBeamAtToken = 19, kBeamAtHyp = 27, kBeamAtRowTok = 43 };
constexpr int kBeamSlotBits = 24;

// Exchange words of one group of 32 workgroups
struct BeamGroupMem {
  unsigned word[96];                              // 0: abort (the session's number), 1: hypotheses written, 32 + g: XCD number of workgroup g
                                                  //   and session, 64 + g: commands done
  unsigned long long cmd[kBeamCmdWords];
  unsigned long long hx[kBeamResHyps * 640];      // new hidden vectors
  unsigned long long px[kBeamResHyps * 640];      // new projections
  unsigned long long ex[kBeamResFrames * 640];    // one scoring step: projected frames
  unsigned long long lg[kBeamResRows * kBeamLgStride];
  unsigned long long row[kBeamResRows * kBeamRowWords];
};
// The scoring step as several launches: where a group's words lie, by the call's sizes.  A launch reads what the one before it wrote, so the
// logits, most of it, need no numbers beside them.  8 groups of 8 hypotheses x 16 frames of 640 units and 1024 labels take 5.5 MB
struct BeamPhaseArea {
  unsigned char *base;
  unsigned px, ex, row, bytes, lg_stride;   // byte offsets inside a group's part (logits: 0) and its size; floats of a row of logits
};
inline BeamPhaseArea beam_phase_area(void *base, int H, int V, int n, int Bh, int K) {
  const unsigned hyps = (unsigned)(Bh + kGroups - 1) / kGroups, rows = hyps * (unsigned)n;
  BeamPhaseArea a{(unsigned char *)base, 0, 0, 0, 0, ((unsigned)V + 32u) / 32u * 32u};
  a.px = (rows * a.lg_stride * 4u + 255u) / 256u * 256u;
  a.ex = a.px + hyps * (unsigned)H * 8u;
  a.row = a.ex + (unsigned)n * (unsigned)H * 8u;
  a.bytes = (a.row + rows * (2u + 2u * (unsigned)K) * 8u + 255u) / 256u * 256u;
  return a;
}
struct BeamResDev {
  const unsigned long long *host_cmd;   // pinned: [kBeamCmdWords]
  unsigned long long *host_res;         // pinned: [kBeamResultWords]
  unsigned *host_exit;                  // pinned: session << 2 | why
  BeamGroupMem *mem;                    // [groups]
  float *h, *c, *p;                     // state slots of the search
  const float *e_all;                   // projected frames
  unsigned session, first;              // number of this launch, and of the first command it takes
  unsigned spin_limit, start_limit;
  unsigned long long idle_ticks;
  // one scoring step (beam_scores_kernel)
  const float *enc, *dec;               // [n, D], [Bh, Hp]
  int n, Bh, K, split;
  int *out_labels, *out_jumps;
  float *out_scores;
  BeamPhaseArea area;                   // as several launches
  unsigned written;                     // hypotheses written by all such launches (BeamGroupMem::word[1] of group 0) once this one is through
};

template <int KS>
struct BeamResCfg {
  static constexpr int H = 128 * KS;                        // = Hp = Hj
  static constexpr int UPW = H / kBeamResWgs, NR = 4 * UPW, LT = NR / 16, PT = (UPW + 15) / 16;   // units and projection rows, tiles of 16 rows
  static constexpr int QK = H / 4, QL = (QK + 63) / 64;     // a wave's quarter of K, and its words per lane
  static constexpr int EST = H + 4;                         // row stride in LDS (16 bytes of padding: banks)
  static constexpr int AST = 12;                            // partial sums of the prediction network: 8 rows, padded
  // command, soft-max rows and merge: behind the rest, in launches of the scoring step ahead of it, some of which need no more
  static constexpr size_t smem_rows = (4 * (kBeamCmdWords + 32 + 2 * 2 * 4 * kBeamResHyps + kBeamResFrames * kBeamRowWords) + 255) / 256 * 256;
  static constexpr size_t oE = 0;                                                   // float [16][EST] frames of the window
  static constexpr size_t oP = oE + (size_t)kBeamResFrames * EST * 4;               // float [16][EST] projections of the hypotheses
  static constexpr size_t oF = oP + (size_t)kBeamPrefixRows * EST * 4;                 // partial sums, one step at a time:
  static constexpr size_t szLogits = (size_t)4 * 3 * 4 * 4 * 80 * 4;                //   float [quarter][tile][row tile][4][80]
  static constexpr size_t oRecp = oF, oPredp = oRecp + (size_t)4 * NR * AST * 4,    //   float [4][NR][AST]; float [4][16 PT][AST]
                          oHst = oPredp + (size_t)4 * 16 * PT * AST * 4;            //   float [8][EST] new hidden vectors
  static constexpr size_t szNet = (size_t)4 * NR * AST * 4 + (size_t)4 * 16 * PT * AST * 4 + (size_t)kBeamResHyps * EST * 4;
  static constexpr size_t szEnc = (size_t)8 * 16 * PT * 20 * 4;                     //   one scoring step: float [8][16 PT][20]
  static constexpr size_t oEncp = oF + szNet;
  static constexpr size_t oI = oF + (szLogits > szNet + szEnc ? szLogits : szNet + szEnc);
  static constexpr size_t smem = oI + smem_rows;
  static_assert(smem <= 160 * 1024, "LDS");
};

// Bounded wait as group_poll, for words that need no clearing between launches: the abort word counts if it holds this session's number
template <class Ask>
__device__ __forceinline__ bool beam_poll(unsigned *abort_word, unsigned session, unsigned limit, const Ask &ask) {
  unsigned spins = 0;
  while (!__all(ask())) {
    if (++spins > limit || ((spins & 15u) == 0 && __hip_atomic_load(abort_word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == session)) {
      if ((threadIdx.x & 63) == 0) __hip_atomic_store(abort_word, session, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      return false;
    }
  }
  return true;
}
__device__ __forceinline__ void beam_st(unsigned long long *p, unsigned lo, unsigned hi) { group_st(p, lo, hi, true); }

// Eight floats as three bf16 vectors that add up to them exactly (24 bits).  FINITE: none is infinite, as the LSTM's own vectors are not; a caller's
// may be: its other two parts are then zero, not what is left of inf - inf, and the products are infinite or NaN as those of fp32 FMA
template <bool FINITE>
__device__ __forceinline__ void beam_split3(const float4 &a, const float4 &b, bf16x8 &hi, bf16x8 &mid, bf16x8 &lo) {
  const float x[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
  u32x4 uh, um, ul;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const float x0 = x[2 * q], x1 = x[2 * q + 1];
    const unsigned h = pack_bf16x2(x0, x1);
    const float h0 = __uint_as_float(h << 16), h1 = __uint_as_float(h & 0xFFFF0000u);
    const float r0 = FINITE || fabsf(h0) != INFINITY ? x0 - h0 : 0.f, r1 = FINITE || fabsf(h1) != INFINITY ? x1 - h1 : 0.f;
    const unsigned d = pack_bf16x2(r0, r1);
    uh[q] = h;
    um[q] = d;
    ul[q] = pack_bf16x2(r0 - __uint_as_float(d << 16), r1 - __uint_as_float(d & 0xFFFF0000u));
  }
  hi = __builtin_bit_cast(bf16x8, uh); mid = __builtin_bit_cast(bf16x8, um); lo = __builtin_bit_cast(bf16x8, ul);
}

// What both forms of the kernel do, per wave; HALF = wave / 4
// PHASES: the scoring step as several launches
template <int KS, int HALF, bool PHASES = false>
struct BeamRes {
  using Cfg = BeamResCfg<KS>;
  static constexpr int H = Cfg::H, QK = Cfg::QK, QL = Cfg::QL, EST = Cfg::EST, NR = Cfg::NR, UPW = Cfg::UPW;
  const ModelDev &m;
  const BeamResDev &r;
  BeamGroupMem &x;               // not PHASES
  unsigned char *const area;     // PHASES: this group's part
  int g, lane, l15, l4, wave, w4, tid;
  float *ecache, *pfull, *fred, *recp, *predp, *hst;
  int *cmd;                      // [kBeamCmdWords] the command; [0] first
  float *s_max, *s_sum, *s_blank;   // [2][4], [2][4], [2]
  int *flags;                    // [4] near, fail
  unsigned *s_wh, *s_wl;         // [2][4][kBeamResHyps]
  unsigned *mrow;                // [kBeamResFrames * kBeamRowWords]
  bool three;                    // this workgroup has the tile of the column past 1023
  static constexpr int LH = HALF == 1 ? (Cfg::LT + 1) / 2 : Cfg::LT / 2, LT0 = HALF == 1 ? 0 : (Cfg::LT + 1) / 2;   // this half's tiles of recurrent rows
  bf16x8 wo[3][KS], wr[LH ? LH : 1][KS], wp[HALF == 0 ? Cfg::PT : 1][KS];
  float bias[3];

  __device__ __forceinline__ unsigned long long *px() const { return PHASES ? reinterpret_cast<unsigned long long *>(area + r.area.px) : x.px; }
  __device__ __forceinline__ unsigned long long *ex() const { return PHASES ? reinterpret_cast<unsigned long long *>(area + r.area.ex) : x.ex; }
  __device__ __forceinline__ unsigned long long *row_words() const { return PHASES ? reinterpret_cast<unsigned long long *>(area + r.area.row) : x.row; }
  __device__ __forceinline__ BeamRes(const ModelDev &m_, const BeamResDev &r_, int grp, unsigned char *smem, int g_)
      : m(m_), r(r_), x(r_.mem[grp]), area(r_.area.base + (size_t)grp * r_.area.bytes), g(g_) {
    tid = threadIdx.x;
    lane = tid & 63; l15 = lane & 15; l4 = lane >> 4;
    wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    w4 = wave & 3;
    unsigned char *const small = smem + (PHASES ? 0 : Cfg::oI);
    if (PHASES) smem += Cfg::smem_rows;
    ecache = reinterpret_cast<float *>(smem + Cfg::oE); pfull = reinterpret_cast<float *>(smem + Cfg::oP);
    fred = reinterpret_cast<float *>(smem + Cfg::oF); recp = reinterpret_cast<float *>(smem + Cfg::oRecp);
    predp = reinterpret_cast<float *>(smem + Cfg::oPredp); hst = reinterpret_cast<float *>(smem + Cfg::oHst);
    cmd = reinterpret_cast<int *>(small);
    s_max = reinterpret_cast<float *>(cmd + kBeamCmdWords); s_sum = s_max + 8; s_blank = s_sum + 8;
    flags = reinterpret_cast<int *>(s_blank + 2);
    s_wh = reinterpret_cast<unsigned *>(cmd + kBeamCmdWords + 32); s_wl = s_wh + 2 * 4 * kBeamResHyps;
    mrow = s_wl + 2 * 4 * kBeamResHyps;
    three = g == kBeamResWgs - 1 && m.V >= 1024;
  }
  __device__ __forceinline__ int tile_col(int t) const { return t == 2 ? 1024 + l15 : 16 * (2 * g + t) + l15; }
  __device__ __forceinline__ void load_w_out() {
#pragma unroll
    for (int t = 0; t < 3; ++t) {
      const bf16_t *src = reinterpret_cast<const bf16_t *>(m.w_out) + (size_t)min(tile_col(t), m.Vpad - 1) * H + w4 * QK + l4 * 8;
#pragma unroll
      for (int i = 0; i < KS; ++i) wo[t][i] = *reinterpret_cast<const bf16x8 *>(src + i * 32);
      bias[t] = m.b_out[min(tile_col(t), m.V)];
    }
  }
  __device__ __forceinline__ void load_w_pred() {
    if constexpr (HALF == 0) {
#pragma unroll
      for (int t = 0; t < Cfg::PT; ++t) {
        const bf16_t *src = reinterpret_cast<const bf16_t *>(m.w_pred) + (size_t)(g * UPW + min(16 * t + l15, UPW - 1)) * H + w4 * QK + l4 * 8;
#pragma unroll
        for (int i = 0; i < KS; ++i) wp[t][i] = *reinterpret_cast<const bf16x8 *>(src + i * 32);
      }
    }
  }
  __device__ __forceinline__ void load_w_rec() {
    if constexpr (LH > 0) {
#pragma unroll
      for (int t = 0; t < LH; ++t) {
        const bf16_t *src = reinterpret_cast<const bf16_t *>(m.w_cat[0]) + (size_t)(g * NR + 16 * (LT0 + t) + l15) * H + w4 * QK + l4 * 8;
#pragma unroll
        for (int i = 0; i < KS; ++i) wr[t][i] = *reinterpret_cast<const bf16x8 *>(src + i * 32);
      }
    }
  }
  __device__ __forceinline__ unsigned *abort_word() const { return &x.word[0]; }
  // A wave that gave up goes on with whatever it holds, but nothing that follows from it is published under the command's number
  template <class Ask>
  __device__ __forceinline__ bool wait(const Ask &ask) const {
    if constexpr (PHASES) { ask(); return true; }   // the launch before wrote them
    const bool got = beam_poll(abort_word(), r.session, r.spin_limit, ask);
    if (!got && lane == 0) flags[1] = 1;
    return got;
  }
  // The number to publish under, once a barrier lies behind the waits of this workgroup
  __device__ __forceinline__ unsigned number(unsigned seq) const { return flags[1] ? 0u : seq; }
  __device__ __forceinline__ unsigned place() const {
    unsigned xcc;
    asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(xcc));
    return (r.session << 4) | (xcc & 15u);
  }
  __device__ __forceinline__ void announce() const {
    if (tid == 0) __hip_atomic_store(&x.word[32 + g], place(), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  // Whether all workgroups of the group are on the chip and share an L2 (wave 0; the result for everybody in flags)
  __device__ __forceinline__ void meet() {
    if (wave == 0) {
      const unsigned mine = place();
      unsigned v = mine;
      const bool got = beam_poll(abort_word(), r.session, r.start_limit, [&]() {
        if (lane < kBeamResWgs) v = __hip_atomic_load(&x.word[32 + lane], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return (v >> 4) == (mine >> 4);
      });
      const bool same = __all(v == mine);
      if (lane == 0) { flags[0] = same; flags[1] = !got; }
    }
    group_barrier();
  }

  // rows of products a x (16 weight rows): fp32 vectors as three bf16 vectors, the small parts in a chain of their own
  template <int T, bool FINITE = true>
  __device__ __forceinline__ void products(const bf16x8 (&w)[T][KS], const float4 (&v)[KS][2], f32x4 (&acc)[T]) const {
    f32x4 small[T];
#pragma unroll
    for (int t = 0; t < T; ++t) acc[t] = small[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < KS; ++i) {
      bf16x8 hi, mid, lo;
      beam_split3<FINITE>(v[i][0], v[i][1], hi, mid, lo);
#pragma unroll
      for (int t = 0; t < T; ++t) {
        small[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(lo, w[t][i], small[t], 0, 0, 0);
        small[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(mid, w[t][i], small[t], 0, 0, 0);
        acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(hi, w[t][i], acc[t], 0, 0, 0);
      }
    }
#pragma unroll
    for (int t = 0; t < T; ++t) acc[t] += small[t];
  }
  // partial sums of rows 0 .. 7 (lanes with l4 < 2) to LDS: [quarter][weight row][AST], this wave's T tiles of N from t0 on
  template <int T, int N>
  __device__ __forceinline__ void put_partial(float *dst, int t0, const f32x4 (&acc)[T]) const {
#pragma unroll
    for (int t = 0; t < T; ++t)
      if (l4 < 2)
        *reinterpret_cast<float4 *>(&dst[((w4 * N + t0 + t) * 16 + l15) * Cfg::AST + 4 * l4]) = make_float4(acc[t][0], acc[t][1], acc[t][2], acc[t][3]);
  }
  __device__ __forceinline__ float sum4(const float *src, int nrows, int row, int e) const {
    float v[4];
#pragma unroll
    for (int w = 0; w < 4; ++w) v[w] = src[(w * nrows + row) * Cfg::AST + e];
    return (v[0] + v[1]) + (v[2] + v[3]);
  }

  // LSTM step and projection of the `fresh` new label sequences of command seq
  __device__ __forceinline__ void network_step(int fresh, unsigned seq) {
    // what a thread's (sequence, gate row) adds to the recurrent sums, and its unit's cell value: asked for ahead of the products
    float add[2], cprev[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int i = min(tid + 512 * q, fresh * NR - 1), e = i / NR, li = i - e * NR;
      add[q] = m.emb_gates[(unsigned)cmd[kBeamAtToken + e] * (4u * H) + (unsigned)(g * NR + li)];
      cprev[q] = r.c[(size_t)cmd[kBeamAtParent + e] * H + g * UPW + (li >> 2)];
    }
    if constexpr (LH > 0) {
      const float *hp = r.h + (size_t)cmd[kBeamAtParent + min(l15, fresh - 1)] * H + w4 * QK + l4 * 8;
      float4 v[KS][2];
#pragma unroll
      for (int i = 0; i < KS; ++i) {
        v[i][0] = *reinterpret_cast<const float4 *>(hp + 32 * i);
        v[i][1] = *reinterpret_cast<const float4 *>(hp + 32 * i + 4);
      }
      f32x4 acc[LH];
      products<LH>(wr, v, acc);
      put_partial<LH, Cfg::LT>(recp, LT0, acc);
    }
    group_barrier();
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int i = tid + 512 * q, e = i / NR, li = i - e * NR;
      if (i < fresh * NR) {   // NR is a multiple of four: a unit's four gates are in one quad, all or none of it
        const float pre = sum4(recp, NR, li, e) + add[q];
        const float act = (li & 3) == 2 ? tanhf(pre) : 1.f / (1.f + expf(-pre));
        const float ig = dpp_f32<0x00>(act), fg = dpp_f32<0x55>(act), gg = dpp_f32<0xAA>(act), og = dpp_f32<0xFF>(act);
        if ((li & 3) == 0) {
          const int u = g * UPW + (li >> 2);
          const size_t at = (size_t)cmd[kBeamAtChild + e] * H + u;
          const float cn = fg * cprev[q] + ig * gg, hn = og * tanhf(cn);
          beam_st(&x.hx[e * H + u], __float_as_uint(hn), seq);
          r.c[at] = cn;
          r.h[at] = hn;
        }
      }
    }
    if constexpr (HALF == 0) {   // this wave's quarter of the new hidden vectors, four sequences at a time
      for (int e0 = 0; e0 < fresh; e0 += 4) {
        unsigned long long u[4][QL];
        wait([&]() {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (e0 + e < fresh) {
#pragma unroll
              for (int q = 0; q < QL; ++q) u[e][q] = group_ld(&x.hx[(e0 + e) * H + w4 * QK + min(lane + 64 * q, QK - 1)]);
            }
          bool now = true;
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (e0 + e < fresh) {
#pragma unroll
              for (int q = 0; q < QL; ++q) now = now && (unsigned)(u[e][q] >> 32) == seq;
            }
          return now;
        });
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (e0 + e < fresh) {
#pragma unroll
            for (int q = 0; q < QL; ++q)
              if (lane + 64 * q < QK) hst[(e0 + e) * EST + w4 * QK + lane + 64 * q] = __uint_as_float((unsigned)u[e][q]);
          }
      }
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // this wave's own part: no barrier
      const float *hp = hst + min(l15, fresh - 1) * EST + w4 * QK + l4 * 8;
      float4 v[KS][2];
#pragma unroll
      for (int i = 0; i < KS; ++i) {
        v[i][0] = *reinterpret_cast<const float4 *>(hp + 32 * i);
        v[i][1] = *reinterpret_cast<const float4 *>(hp + 32 * i + 4);
      }
      f32x4 acc[Cfg::PT];
      products<Cfg::PT>(wp, v, acc);
      put_partial<Cfg::PT, Cfg::PT>(predp, 0, acc);
    }
    group_barrier();
    if (tid < fresh * UPW) {
      const int e = tid / UPW, row = tid - e * UPW;
      const float v = sum4(predp, 16 * Cfg::PT, row, e) + m.b_pred[g * UPW + row];
      beam_st(&x.px[e * H + g * UPW + row], __float_as_uint(v), number(seq));
      r.p[(size_t)cmd[kBeamAtChild + e] * H + g * UPW + row] = v;
    }
  }

  // Projections of the command's hypotheses into LDS: a half takes every other one, a wave its quarter
  __device__ __forceinline__ void fetch_projections(int Bh, unsigned seq) {
    for (int b0 = HALF; b0 < Bh; b0 += 8) {
      unsigned long long u[4][QL];
      int word[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) word[e] = __builtin_amdgcn_readfirstlane(cmd[kBeamAtHyp + min(b0 + 2 * e, Bh - 1)]);
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if ((unsigned)word[e] >> kBeamSlotBits == 0u) {
#pragma unroll
          for (int q = 0; q < QL; ++q)
            u[e][q] = ((unsigned long long)seq << 32) | __float_as_uint(r.p[(size_t)word[e] * H + w4 * QK + min(lane + 64 * q, QK - 1)]);
        }
      wait([&]() {
        bool now = true;
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if ((unsigned)word[e] >> kBeamSlotBits) {
#pragma unroll
            for (int q = 0; q < QL; ++q)
              u[e][q] = group_ld(&x.px[(((unsigned)word[e] >> kBeamSlotBits) - 1u) * H + w4 * QK + min(lane + 64 * q, QK - 1)]);
          }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
#pragma unroll
          for (int q = 0; q < QL; ++q) now = now && (unsigned)(u[e][q] >> 32) == seq;
        }
        return now;
      });
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (b0 + 2 * e < Bh) {
#pragma unroll
          for (int q = 0; q < QL; ++q)
            if (lane + 64 * q < QK) pfull[(b0 + 2 * e) * EST + w4 * QK + lane + 64 * q] = __uint_as_float((unsigned)u[e][q]);
        }
    }
  }

  // Logits of rows (hypothesis b, frame j), row = b n + j, this workgroup's columns, as words for whoever needs them.  Ends in a barrier.
  __device__ __forceinline__ void logits(int rows, int n, int split, unsigned seq) {
    const unsigned ninv = 65536u / (unsigned)n + 1u;   // x / n for x < 128
    const unsigned num = number(seq);
    for (int r0 = 0; r0 < rows; r0 += 64) {
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const int rt = HALF + 2 * q;
        if (r0 + 16 * rt >= rows) continue;
        const int row = min(r0 + 16 * rt + l15, rows - 1), b = (int)(((unsigned)row * ninv) >> 16), j = row - b * n;
        const float *er = ecache + j * EST + w4 * QK + l4 * 8, *pr = pfull + b * EST + w4 * QK + l4 * 8;
        f32x4 acc[3];
#pragma unroll
        for (int t = 0; t < 3; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < KS; ++i) {
          float z[8];
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            const float4 e4 = *reinterpret_cast<const float4 *>(er + i * 32 + 4 * h), p4 = *reinterpret_cast<const float4 *>(pr + i * 32 + 4 * h);
            z[4 * h + 0] = fmaxf(e4.x + p4.x, 0.f); z[4 * h + 1] = fmaxf(e4.y + p4.y, 0.f);
            z[4 * h + 2] = fmaxf(e4.z + p4.z, 0.f); z[4 * h + 3] = fmaxf(e4.w + p4.w, 0.f);
          }
          u32x4 zu, zl;
#pragma unroll
          for (int h = 0; h < 4; ++h) {
            zu[h] = pack_bf16x2(z[2 * h], z[2 * h + 1]);
            zl[h] = pack_bf16x2(z[2 * h] - __uint_as_float(zu[h] << 16), z[2 * h + 1] - __uint_as_float(zu[h] & 0xFFFF0000u));
          }
          const bf16x8 zh = __builtin_bit_cast(bf16x8, zu), zr = __builtin_bit_cast(bf16x8, zl);
#pragma unroll
          for (int t = 0; t < 3; ++t)
            if (t < 2 || three) {
              acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(zh, wo[t][i], acc[t], 0, 0, 0);
              if (split) acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(zr, wo[t][i], acc[t], 0, 0, 0);
            }
        }
#pragma unroll
        for (int t = 0; t < 3; ++t)
#pragma unroll
          for (int k = 0; k < 4; ++k) fred[(((w4 * 3 + t) * 4 + rt) * 4 + k) * 80 + lane] = acc[t][k];
      }
      group_barrier();
      // register k of lane l: row 4 l4 + k of the tile, column l15: one (row tile, k, column tile) per wave and turn
      auto finish = [&](int rt, int k, int t) {
        const int row = r0 + 16 * rt + 4 * l4 + k, col = tile_col(t);
        float v[4];
#pragma unroll
        for (int w = 0; w < 4; ++w) v[w] = fred[(((w * 3 + t) * 4 + rt) * 4 + k) * 80 + lane];
        const float logit = (v[0] + v[1]) + (v[2] + v[3]) + (t == 0 ? bias[0] : t == 1 ? bias[1] : bias[2]);
        if (row < rows && col <= m.V) {
          if constexpr (PHASES) reinterpret_cast<float *>(area)[(unsigned)row * r.area.lg_stride + (unsigned)col] = logit;
          else beam_st(&x.lg[row * kBeamLgStride + col], __float_as_uint(logit), num);
        }
      };
#pragma unroll
      for (int q = 0; q < 4; ++q) finish(wave & 3, q, HALF);
      if (three) {
#pragma unroll
        for (int q = 0; q < 2; ++q) finish(wave & 3, 2 * HALF + q, 2);
      }
      group_barrier();
    }
  }

  // Soft-max of rows g, g + 32, ... (a half takes every other one), and the K largest label logits of each, for the merge;
  // or (complete) log soft-max of the row's own label, straight to the host
  __device__ __forceinline__ void soft_max_rows(int rows, int K, bool complete, unsigned seq) {
    constexpr int EPT = 5;   // 1025 entries over four waves
    const int V = m.V, rounds = rows > g ? (rows - g + 2 * kBeamResWgs - 1) / (2 * kBeamResWgs) : 0;
    for (int q = 0; q < rounds; ++q) {
      const int row = g + kBeamResWgs * (2 * q + HALF);
      const bool mine = row < rows;
      const int v0 = w4 * 64 + lane;
      if (mine) {
        unsigned long long u[EPT];
        wait([&]() {
          bool now = true;
#pragma unroll
          for (int i = 0; i < EPT; ++i) {
            const int v = min(v0 + 256 * i, V);
            if constexpr (PHASES) u[i] = __float_as_uint(reinterpret_cast<const float *>(area)[(unsigned)row * r.area.lg_stride + (unsigned)v]);
            else u[i] = group_ld(&x.lg[row * kBeamLgStride + v]);
          }
#pragma unroll
          for (int i = 0; i < EPT; ++i) now = now && (unsigned)(u[i] >> 32) == seq;
          return now;
        });
        float a[EPT];
#pragma unroll
        for (int i = 0; i < EPT; ++i) a[i] = v0 + 256 * i <= V ? __uint_as_float((unsigned)u[i]) : -INFINITY;
        float mx = a[0];
#pragma unroll
        for (int i = 1; i < EPT; ++i) mx = fmaxf(mx, a[i]);
        mx = wave_max_f32(mx);
        float sum = 0.f;
        if (mx > -INFINITY) {
#pragma unroll
          for (int i = 0; i < EPT; ++i) sum += expf(a[i] - mx);
        }
        sum = wave_sum(sum);
        if (lane == 0) { s_max[HALF * 4 + w4] = mx; s_sum[HALF * 4 + w4] = sum; }
        const int special = complete ? cmd[kBeamAtRowTok + min(row, kBeamPrefixRows - 1)] : V;   // the entry whose log-probability is wanted
#pragma unroll
        for (int i = 0; i < EPT; ++i)
          if (v0 + 256 * i == special) s_blank[HALF] = a[i];
        if (!complete) {
          // K rounds of "largest remaining label entry of my 64 lanes"; lane k keeps the k-th
          unsigned hi[EPT], win_h = 0u, win_l = 0u;
#pragma unroll
          for (int i = 0; i < EPT; ++i) hi[i] = v0 + 256 * i < V ? beam_order_bits(a[i]) : 0u;
          for (int k = 0; k < K; ++k) {
            unsigned bh = 0u, bl = 0u;
#pragma unroll
            for (int i = 0; i < EPT; ++i) {   // labels rise with i: an equal later one does not win
              const bool better = hi[i] > bh;
              bh = better ? hi[i] : bh;
              bl = better ? ~(unsigned)(v0 + 256 * i) : bl;
            }
            wave_max_pair(bh, bl);
            const int v = (int)~bl;
            if (bh != 0u && (v & 255) == v0) {   // its owner retires it
#pragma unroll
              for (int i = 0; i < EPT; ++i)
                if (i == (v >> 8)) hi[i] = 0u;
            }
            if (lane == k) { win_h = bh; win_l = bl; }
          }
          if (lane < K) { s_wh[(HALF * 4 + w4) * kBeamResHyps + lane] = win_h; s_wl[(HALF * 4 + w4) * kBeamResHyps + lane] = win_l; }
        }
      }
      group_barrier();
      const unsigned num = number(seq);
      if (mine && w4 == 0 && num) {
        const float *pm = s_max + HALF * 4, *ps = s_sum + HALF * 4;
        const float mx = fmaxf(fmaxf(pm[0], pm[1]), fmaxf(pm[2], pm[3]));
        float sum = 0.f;
#pragma unroll
        for (int w = 0; w < 4; ++w) sum += ps[w] * expf(pm[w] - mx);
        const float lse = mx + logf(sum), special = s_blank[HALF] - lse;
        if (complete) {
          if (lane == 0) __hip_atomic_store(r.host_res + row, (unsigned long long)__float_as_uint(special) | ((unsigned long long)(seq | 0x80000000u) << 32), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        } else {
          int head = 0;   // lanes 0..3: head of wave `lane`'s list
          unsigned res_h = 0u, res_l = 0u;
          const unsigned *lh = s_wh + (HALF * 4 + (lane & 3)) * kBeamResHyps, *ll = s_wl + (HALF * 4 + (lane & 3)) * kBeamResHyps;
          for (int k = 0; k < K; ++k) {
            unsigned h = (lane < 4 && head < K) ? lh[head] : 0u, l = (lane < 4 && head < K) ? ll[head] : 0u;
            const unsigned myh = h, myl = l;
            wave_max_pair<16>(h, l);   // K <= 8: heads and winners are in the first row of lanes
            if (lane < 4 && myh == h && myl == l && h != 0u) ++head;
            if (lane == k) { res_h = h; res_l = l; }
          }
          unsigned long long *out = row_words() + row * (2 + 2 * K);
          if (lane < K) {
            beam_st(out + 2 + 2 * lane, res_h != 0u ? __float_as_uint(beam_score_of(res_h)) : __float_as_uint(-INFINITY), seq);
            beam_st(out + 3 + 2 * lane, res_h != 0u ? ~res_l : ~0u, seq);
          }
          if (lane == 0) {
            beam_st(out, __float_as_uint(lse), seq);
            beam_st(out + 1, __float_as_uint(special), seq);
          }
        }
      }
      if (q + 1 < rounds) group_barrier();
    }
  }

  // One wave: the K best pairs of hypothesis b (its n rows' candidates; beam_merge_kernel's rules).  Lane k is handed the k-th.
  template <class Put>
  __device__ __forceinline__ void merge(int b, int n, int K, unsigned seq, const Put &put) {
    const int RW = 2 + 2 * K, total = n * RW, V1 = m.V + 1;
    constexpr int NQ = (kBeamResFrames * kBeamRowWords + 63) / 64;
    const unsigned long long *src = row_words() + (size_t)b * n * RW;
    unsigned long long u[NQ];
    const bool got = wait([&]() {
      bool now = true;
#pragma unroll
      for (int q = 0; q < NQ; ++q) u[q] = group_ld(src + min(lane + 64 * q, total - 1));
#pragma unroll
      for (int q = 0; q < NQ; ++q) now = now && (unsigned)(u[q] >> 32) == seq;
      return now;
    });
#pragma unroll
    for (int q = 0; q < NQ; ++q)
      if (lane + 64 * q < total) mrow[lane + 64 * q] = (unsigned)u[q];
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    const bool has_row = lane < n;
    const unsigned *mine = mrow + (has_row ? lane : 0) * RW;
    const float my_blank = has_row ? __uint_as_float(mine[1]) : 0.f;
    float run = 0.f, all = 0.f;
    for (int t = 0; t < n; ++t) {
      const float v = readlane_f32(my_blank, t);
      if (lane == t) run = all;
      all += v;
    }
    const float add = has_row ? run - __uint_as_float(mine[0]) : 0.f;
    unsigned blank_h = beam_order_bits(all), blank_l = ~(unsigned)((n - 1) * V1 + m.V), res_h = 0u, res_l = 0u;
    int head = 0;
    float cur = __uint_as_float(mine[2]);
    int curv = has_row ? (int)mine[3] : -1;
    for (int k = 0; k < K; ++k) {
      unsigned h = 0u, l = 0u;
      if (head < K && curv >= 0) { h = beam_order_bits(cur + add); l = ~(unsigned)(lane * V1 + curv); }
      const unsigned myh = h, myl = l;
      wave_max_pair<16>(h, l);   // n <= 16 rows, K <= 8 winners: the first row of lanes
      if (blank_h != 0u && (blank_h > h || (blank_h == h && blank_l > l))) { h = blank_h; l = blank_l; blank_h = 0u; }
      else if (myh == h && myl == l && h != 0u) {
        ++head;
        cur = __uint_as_float(mine[2 + 2 * min(head, K - 1)]);
        curv = (int)mine[3 + 2 * min(head, K - 1)];
      }
      if (lane == k) { res_h = h; res_l = l; }
    }
    const int key = (int)~res_l;
    if (lane < K && got) put(lane, res_h != 0u, key % V1, key / V1, res_h != 0u ? beam_score_of(res_h) : -INFINITY);
  }

  __device__ __forceinline__ void search() {
    announce();
    load_w_out();
    load_w_pred();
    load_w_rec();
    meet();
    unsigned why = kBeamExitFailed;   // of wave 0 of workgroup 0
    bool failed = !flags[0] || flags[1];
    for (unsigned seq = r.first; !failed; ++seq) {
      // opaque: what follows from the lane's number is formed again where it is used, not kept in registers that the weights need
      asm volatile("" : "+v"(lane), "+v"(tid));
      l15 = lane & 15;
      l4 = lane >> 4;
      if (wave == 0) {
        unsigned u = kBeamCmdQuit;
        why = kBeamExitFailed;
        if (g == 0) {
          bool go = seq == r.first || beam_poll(abort_word(), r.session, r.spin_limit, [&]() {   // everybody is done with the last one
            return lane >= kBeamResWgs || __hip_atomic_load(&x.word[64 + lane], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == seq - 1u;
          });
          const unsigned long long t0 = wall_clock64();
          while (go) {
            const unsigned gone = __hip_atomic_load(abort_word(), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const unsigned long long w = __hip_atomic_load(r.host_cmd + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
            if (__all((unsigned)(w >> 32) == seq)) {
              u = (unsigned)w;
              why = kBeamExitAsked;
              break;
            }
            const bool moved_on = __any((unsigned)(w >> 32) == seq + 1u);   // this one asked to leave, and the next, for another launch, is there already
            const bool idle = wall_clock64() - t0 > r.idle_ticks;
            why = moved_on ? kBeamExitAsked : idle ? kBeamExitIdle : kBeamExitFailed;
            go = !moved_on && !idle && gone != r.session;
          }
          beam_st(&x.cmd[lane], u, seq);
        } else {
          unsigned long long w = 0ull;
          if (beam_poll(abort_word(), r.session, r.spin_limit, [&]() { w = group_ld(&x.cmd[lane]); return (unsigned)(w >> 32) == seq; })) u = (unsigned)w;
        }
        cmd[lane] = (int)u;
      }
      group_barrier();
      const int head = __builtin_amdgcn_readfirstlane(cmd[kBeamAtHead]), kind = head & 0xFF, fresh = (head >> 8) & 0xFF, Bh = (head >> 16) & 0xFF, n = head >> 24;
      const int t = __builtin_amdgcn_readfirstlane(cmd[kBeamAtFrame]), kw = __builtin_amdgcn_readfirstlane(cmd[kBeamAtK]), K = kw & 0xFF, split = kw >> 8;
      if (kind == kBeamCmdQuit) break;
      // the window's projected frames: a frame per wave, straight to LDS, looked at behind the projections' exchange
      const unsigned lds0 = (unsigned)(unsigned long long)(__attribute__((address_space(3))) const float *)ecache;
      for (int f = wave; f < n; f += 8) {
#pragma unroll
        for (int i = 0; i < (H + 255) / 256; ++i)
          if (i * 256 + lane * 4 < H) group_load_lds(r.e_all + (size_t)(t + f) * H + i * 256 + lane * 4, lds0 + (unsigned)f * (EST * 4) + i * 1024);
      }
      if (fresh) network_step(fresh, seq);
      fetch_projections(Bh, seq);
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      group_barrier();
      const int rows = Bh * n;
      logits(rows, n, split, seq);
      soft_max_rows(rows, K, kind == kBeamCmdComplete, seq);
      if (kind == kBeamCmdScore && HALF == 1 && w4 == 1 && g < Bh) {
        const unsigned tag = (seq & 0x7FFFu) | 0x8000u;
        merge(g, n, K, seq, [&](int k, bool any, int label, int jump, float score) {
          const unsigned code = any ? (unsigned)(jump << 11 | label) : (unsigned)kBeamCodeNone;
          __hip_atomic_store(r.host_res + g * K + k, (unsigned long long)__float_as_uint(score) | ((unsigned long long)(tag << 16 | code) << 32), __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_SYSTEM);
        });
      }
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // what this command wrote has reached the L2
      group_barrier();
      failed = flags[1];
      if (tid == 0) group_publish(&x.word[64 + g], seq, true);
      group_barrier();   // everybody has looked at the flag, nobody reads this command any more
    }
    if (g == 0 && tid == 0) {
      if (failed) why = kBeamExitFailed;
      __hip_atomic_store(r.host_exit, r.session << 2 | why, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
  }

  // Rows of words (H each) into LDS: a half takes every other row, a wave its quarter
  __device__ __forceinline__ void fetch_rows(const unsigned long long *src, float *dst, int count, unsigned seq) {
    for (int b0 = HALF; b0 < count; b0 += 8) {
      unsigned long long u[4][QL];
      wait([&]() {
        bool now = true;
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int q = 0; q < QL; ++q) u[e][q] = group_ld(src + min(b0 + 2 * e, count - 1) * H + w4 * QK + min(lane + 64 * q, QK - 1));
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int q = 0; q < QL; ++q) now = now && (unsigned)(u[e][q] >> 32) == seq;
        return now;
      });
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (b0 + 2 * e < count) {
#pragma unroll
          for (int q = 0; q < QL; ++q)
            if (lane + 64 * q < QK) dst[(b0 + 2 * e) * EST + w4 * QK + lane + 64 * q] = __uint_as_float((unsigned)u[e][q]);
        }
    }
  }

  // One scoring step: group grp takes hypotheses grp, grp + kGroups, ...  Its workgroups project the window's frames and those hypotheses
  // (every group all the frames: 26 MFLOP, less than telling the other XCDs), each its units, and go on as in a pass of the search.
  // PHASE 0 to 3: the same in four launches, each up to an exchange and then the next, for calls that nobody waits for: every word is there
  // when it is asked for, no two workgroups have to meet, and every sum is the one launch's, to the bit
  template <int PHASE>
  __device__ __forceinline__ void score(int grp) {
    const unsigned seq = r.first;
    const int n = r.n, Bg = (r.Bh - grp + kGroups - 1) / kGroups, D = m.D, u0 = g * UPW;
    float *encp = reinterpret_cast<float *>(reinterpret_cast<unsigned char *>(ecache) + (Cfg::oEncp - Cfg::oE));
    if constexpr (PHASE < 0) {
      announce();
    } else {
      if (tid == 0) { flags[0] = 1; flags[1] = 0; }
      group_barrier();
    }
    if constexpr (PHASE <= 0) {
    // Everything the launch reads is asked for before any of it is looked at (start to the projections 8.9 -> 8.2 us).  Frames: K split over the
    // eight waves in steps of 32, four at a time; rounded to bf16 as everywhere in bf16 models
    f32x4 acc[Cfg::PT];
#pragma unroll
    for (int t = 0; t < Cfg::PT; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
    const float *er = r.enc + (size_t)min(l15, n - 1) * D + l4 * 8;
    const bf16_t *wr0 = reinterpret_cast<const bf16_t *>(m.w_enc) + l4 * 8;
    float4 ea[4], eb[4];
    bf16x8 we[4][Cfg::PT];
    auto ask_frames = [&](int k0) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int k = min(k0 + 256 * q, D - 32);
        ea[q] = *reinterpret_cast<const float4 *>(er + k);
        eb[q] = *reinterpret_cast<const float4 *>(er + k + 4);
#pragma unroll
        for (int t = 0; t < Cfg::PT; ++t) we[q][t] = *reinterpret_cast<const bf16x8 *>(wr0 + (size_t)(u0 + min(16 * t + l15, UPW - 1)) * D + k);
      }
    };
    ask_frames(wave * 32);
    float4 v[KS][2];
    if constexpr (HALF == 0) {
      const float *hp = r.dec + (size_t)(grp + kGroups * min(l15, Bg - 1)) * H + w4 * QK + l4 * 8;
#pragma unroll
      for (int i = 0; i < KS; ++i) {
        v[i][0] = *reinterpret_cast<const float4 *>(hp + 32 * i);
        v[i][1] = *reinterpret_cast<const float4 *>(hp + 32 * i + 4);
      }
    }
    load_w_pred();
    if constexpr (PHASE < 0) load_w_out();
    __builtin_amdgcn_sched_barrier(0);
    for (int k0 = wave * 32; k0 < D; k0 += 1024) {
      if (k0 >= 1024) ask_frames(k0);
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (k0 + 256 * q < D) {
          const u32x4 xu = u32x4{pack_bf16x2(ea[q].x, ea[q].y), pack_bf16x2(ea[q].z, ea[q].w), pack_bf16x2(eb[q].x, eb[q].y), pack_bf16x2(eb[q].z, eb[q].w)};
#pragma unroll
          for (int t = 0; t < Cfg::PT; ++t) acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, xu), we[q][t], acc[t], 0, 0, 0);
        }
    }
#pragma unroll
    for (int t = 0; t < Cfg::PT; ++t)
      *reinterpret_cast<float4 *>(&encp[((wave * Cfg::PT + t) * 16 + l15) * 20 + 4 * l4]) = make_float4(acc[t][0], acc[t][1], acc[t][2], acc[t][3]);
    if constexpr (HALF == 0) {
      f32x4 pacc[Cfg::PT];
      products<Cfg::PT, false>(wp, v, pacc);
      put_partial<Cfg::PT, Cfg::PT>(predp, 0, pacc);
    }
    if constexpr (PHASE < 0) meet();   // a barrier: the partial sums are in LDS
    else group_barrier();
    if (!flags[0] || flags[1]) return;
    for (int i = tid; i < (n + Bg) * UPW; i += 512) {
      const int e = i / UPW, row = i - e * UPW;
      if (e < n) {
        float v[8];
#pragma unroll
        for (int w = 0; w < 8; ++w) v[w] = encp[(w * 16 * Cfg::PT + row) * 20 + e];
        beam_st(ex() + e * H + u0 + row, __float_as_uint(((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7])) + m.b_enc[u0 + row]), seq);
      } else {
        beam_st(px() + (e - n) * H + u0 + row, __float_as_uint(sum4(predp, 16 * Cfg::PT, row, e - n) + m.b_pred[u0 + row]), seq);
      }
    }
    }
    if constexpr (PHASE == 0) return;
    // No wait of this launch may outlast its results, the words are the next one's then: whoever has no part in them leaves
    if (PHASE < 0 && 32 * g > m.V && g >= Bg * n) return;   // no column, no row
    if constexpr (PHASE < 0 || PHASE == 1) {
      if constexpr (PHASE == 1) load_w_out();
      fetch_rows(ex(), ecache, n, seq);
      fetch_rows(px(), pfull, Bg, seq);
      group_barrier();
      logits(Bg * n, n, r.split, seq);
    }
    if constexpr (PHASE < 0 || PHASE == 2) soft_max_rows(Bg * n, r.K, false, seq);
    if constexpr (PHASE == 1 || PHASE == 2) return;
    if (HALF == 1 && w4 == 1 && g < Bg) {
      const int b = grp + kGroups * g;
      bool put = false;
      merge(g, n, r.K, seq, [&](int k, bool any, int label, int jump, float score) {
        const size_t o = (size_t)b * r.K + k;
        __hip_atomic_store(r.out_labels + o, any ? label : -1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(r.out_jumps + o, any ? jump : -1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(r.out_scores + o, score, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        put = true;
      });
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // they are in memory: the last hypothesis of the launch tells the host
      if (PHASE < 0 && put && lane == 0 && __hip_atomic_fetch_add(&r.mem[0].word[1], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1u == r.written)
        __hip_atomic_store(r.host_exit, r.session << 2 | kBeamExitAsked, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
  }
};

template <int KS>
__global__ __launch_bounds__(512) void beam_search_kernel(ModelDev m, BeamResDev r) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem_raw[];
  if (blockIdx.x % kGroups != 0) return;   // workgroups go to the XCDs in turn
  const int g = (int)blockIdx.x / kGroups;
  if (threadIdx.x < 256) BeamRes<KS, 0>(m, r, 0, smem_raw, g).search();
  else BeamRes<KS, 1>(m, r, 0, smem_raw, g).search();
}

// One scoring step for up to 64 hypotheses and 16 frames, a group of workgroups per XCD, a single launch.  As five launches (two
// projections, logits, rows, merge) and a wait for the stream 16 hypotheses x 16 frames of 640 units and 1024 labels took 54 us, now 35.5: 20 in the kernel
// (memory to projections 8.2, exchange and frames to LDS 3, logits 2, rows, merge and their exchanges 7), the rest launch and return.
template <int KS>
__global__ __launch_bounds__(512) void beam_scores_kernel(ModelDev m, BeamResDev r) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem_raw[];
  const int grp = (int)blockIdx.x % kGroups, g = (int)blockIdx.x / kGroups;
  if (grp >= r.Bh) return;
  if (threadIdx.x < 256) BeamRes<KS, 0>(m, r, grp, smem_raw, g).template score<-1>(grp);
  else BeamRes<KS, 1>(m, r, grp, smem_raw, g).template score<-1>(grp);
}
template <int KS, int PHASE>
__global__ __launch_bounds__(512) void beam_scores_phase_kernel(ModelDev m, BeamResDev r) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem_raw[];
  const int grp = (int)blockIdx.x % kGroups, g = (int)blockIdx.x / kGroups;
  if (grp >= r.Bh) return;
  if (threadIdx.x < 256) BeamRes<KS, 0, true>(m, r, grp, smem_raw, g).template score<PHASE>(grp);
  else BeamRes<KS, 1, true>(m, r, grp, smem_raw, g).template score<PHASE>(grp);
}

}  // namespace wind
