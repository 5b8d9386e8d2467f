// The whole decode loop of batches of models with larger vocabularies as resident groups of workgroups, one group per XCD.
#pragma once
#include "wind_types.h"
#include "wind_decide_kernels.h"
#include "wind_group_kernel.h"
#include "wind_group_protocol.h"

namespace wind {

// ---------------------------------------------------------------------------------------------
// Like wind_group_kernel, for 993 to 4096 labels and up to 32 utterances per group at a time, each in a slot of its own from the first to
// the last frame.  There every workgroup forms every window row and takes every slot's decision, which with 32 slots and 128 key
// parts would be all that it did; here the work is cut so that none is done twice:
//   z     workgroup g holds PPW columns of W_pred and of the joint hidden vector: it adds its columns of the window's projected frames (LDS) and
//         of the slots' projections (its own sums), applies the ReLU and rounds: its columns of every window row, and its part of the
//         row's blank logit and squared norm                                                        -> exchange z (fp16), bn (fp32)
//   keys  it fetches all window rows, in chunks of 32, through registers (waves 4-7) into LDS, and multiplies them (waves 0-3, each a part
//         of 32 columns over the whole of K, weights in registers, the transposed product: a lane holds 16 logits of one row)
//                                                                                                   -> exchange keys
//   step  workgroup s decides slot s (its keys, near-ties in fp32)                                  -> exchange dec
//   h     everybody takes the LSTM step of its units for all slots with a label                     -> exchange h (bf16, high and low part)
//         and forms the projection columns of the new hidden vectors (waves 4-7, K split in four; the recurrent sums of the next
//         step likewise, beside the decisions)
// What bounds it: the chain of four exchanges through the group's L2 (0.6 to 1 us each) and the label's row of input gate
// sums from memory; with many slots the products and the rows' way through LDS (a chunk of 32 rows 1.05 us: 0.6 of products, whose rows come from LDS at
// the 128 bytes per clock that it gives).  640 units, 4096 labels, us per iteration, 6 / 32 slots: z 0.8 / 1.5, first chunk in LDS
// 0.8 / 0.3, products 1.2 / 4.4, decision 1.6 / 2.2, its word and the slots' states 1.0 / 1.6, LSTM step 1.1 / 1.9, hidden vectors and projection 1.5 / 2.5.
// Whole decodes of up to 1000 frames, W = 16, per-step kernels (four launches, 22 to 30 us per iteration) / groups: a label on every second evaluation,
// 8 utterances 18.1 / 5.4 ms, 45 21.9 / 6.5, 128 26.8 / 8.8, 256 29.8 / 11.0; hardly any label 8 utterances 1.42 / 0.53, 64 2.1 / 0.89, 128 2.4 / 1.19, 256 3.2 / 2.0.
// Tried: waves 4-7 form every other 256 items of the window rows (32 slots: 0.3 us less there, 0.5 more until the first chunk, whose fetching waits for
// the recurrent sums behind that); the deciding wave brings its label's row of input sums into the L2 ahead of the step: what the asking took it (0.6 us) was more than
// the step gained; a wave per quad for windows of one quad too (18 words per lane instead of 5): 0.8 us slower.
//
// Rows of a window: quads of 4, one to `qmax` per slot: a window without a label doubles its slot's next one, a label takes it back, so
// that rows behind labels are not computed and stretches of blanks go by in long steps.  With few slots longer windows to begin with (16 rows for up to
// two, 8 for up to four, all in one chunk of products) take fewer iterations and a slower decision: 8 utterances, a label on every second evaluation 5.86 / 5.26 ms,
// 24 5.56 / 5.21; hardly any label 0.50 / 0.52.  A quad of z holds, per 4 columns, its 4 rows' words of 8
// bytes: what a workgroup writes and what a wave fetches are whole segments.
//
// No barrier between workgroups and no flag words: every word tells whether it is the one that is waited for.  z has a free sign bit
// (the ReLU's results), h a free exponent bit (|h| <= 1), keys and norms a bit of their mantissa; these alternate from one use of a row
// (h: from one step of the slot, in two buffers) to the next.  dec and the projections' words carry the iteration or step number.  No word is overwritten
// before everybody has read it:
//   z, bn, keys of a row   are written after its slot's last decision, which its owner took from everybody's keys of the row's last use, which
//                          were formed from the z before (every workgroup has a key part: more labels than 31 parts)
//   dec                    is written after everybody's keys of this iteration, so after everybody's barrier behind the last dec
//   h                      of a step: everybody reads it for the projection and, up to the next decision, for the recurrent sums; it is
//                          overwritten two steps of the slot later
// Waits are bounded as in wind_group_kernel.
//
// Registers: the weights of 640 units fill them: nine vector registers (40 bytes per lane) lie in scratch memory there, none with fewer units, and 78 to 143
// scalars in lanes of vector registers.
constexpr int kVocabSlots = 32;
constexpr int kTie = 0x3FFF;   // instead of a label: a near-tie
// The screening products are fp16: as fast as bf16 and with eight times less rounding of the hidden row, so that near-ties, each of which holds all
// slots up for 2 us, are eight times rarer (one iteration in eight with 16 slots instead of two in three).  The weights are scaled by a power of two that
// makes the largest about 2^14 (ModelDev::w16_scale), which keeps what fp16 cannot hold of them in full far below the rounding of the rest; the rows are not:
// fp16 holds units of up to 65504, and the products take its smallest numbers as they are.  Rows longer than kZ16Max, where a unit might not fit, leave the call to the
// per-step kernels at once (as groups that cannot meet do): 640 units, 4096 labels, every row such, 8 / 128 utterances of up to 100 frames 3.09 / 4.19 ms, with those kernels
// from the start 2.95 / 4.04, where rows that fit take 0.97 / 1.43.  (Decided over all labels in fp32 by one wave, at lengths above 1000: 191 / 527 ms.)
// Rows decided again, 256 utterances of 640 units and 4096 labels: 9283 with bf16, now 1311; 11.4 -> 11.0 ms, 45 utterances 6.61 -> 6.42, 8 5.94 -> 5.87.
constexpr float kZ16Max = 64000.f;
// A row's squared norm is exchanged in parts of four units.  Their sums stay below kNormInfinite where all units are finite, also where squares overflow, and
// with an infinite unit they do not (a word's lowest bit is its tag: no infinity).
constexpr float kNormPart = 1e35f, kNormInfinite = 1e38f;
typedef __attribute__((ext_vector_type(8))) _Float16 f16x8;
typedef __attribute__((ext_vector_type(2))) _Float16 f16x2_t;
__device__ __forceinline__ uint32_t pack_f16x2(float lo, float hi) {
  const f32x2_t v = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, f16x2_t));
}
// How far below the best a label may be to be looked at in fp32: see decide_row; an eighth of bf16's rounding, and what fp16's smallest numbers lose
__device__ __forceinline__ float vocab_band(const ModelDev &m, float znorm, float top) {
  return fmaf(m.tau_scale * 0.125f, znorm, m.tau16_floor) + 6.2e-5f * fabsf(top);
}

template <int KS>
struct VocabCfg {
  static constexpr int GW = 32, H = 128 * KS, UPW = H / GW, NR = 4 * UPW, PPW = H / GW;
  static constexpr int LT = NR / 16, PT = (PPW + 15) / 16;
  static constexpr int QK = H / 4;
  static constexpr int ZST = H + 8;                                            // fp16 per row in LDS (16 bytes of padding: banks)
  static constexpr int NC = PPW / 4;                                           // groups of 4 columns
  static constexpr size_t oZ = 0;                                              // fp16 [2][32][ZST]; between them the partial sums of the recurrent rows, float [4][32][NR]
  static constexpr size_t kZBuf = (size_t)32 * ZST * 2;
  static constexpr size_t oE = oZ + 2 * kZBuf;                                 // float4 [NC][512]: slot x ring
  static constexpr size_t oPred = oE + (size_t)NC * 512 * 16;                  // float [4][32][PPW]
  static constexpr size_t oP = oPred + (size_t)4 * kVocabSlots * PPW * 4;      // float [32][PPW]
  static constexpr size_t oRec = oP + (size_t)kVocabSlots * PPW * 4;           // float [32][NR]
  static constexpr size_t oC = oRec + (size_t)kVocabSlots * NR * 4;            // float [32][UPW]
  static constexpr size_t oPf = oC + (size_t)kVocabSlots * UPW * 4;            // float [H] projection of this workgroup's own slot
  static constexpr size_t oB = oPf + (size_t)H * 4;                            // float [4][32] output biases
  static constexpr size_t oWb = oB + 512;                                      // float [PPW] blank column, [PPW] projection biases
  static constexpr size_t oS = oWb + (size_t)2 * PPW * 4;                      // VocabSlot [2][32], of this iteration and of the next
  static constexpr size_t oQ = oS + 2 * kVocabSlots * 32;                      // int [64] quads of the iteration
  static constexpr size_t oI = oQ + 64 * 4;                                    // int info[32], emap[2][32], stat[16], rech[16], head[4], counts[kNumStats + 2], fail, near
  static constexpr size_t smem = oI + (size_t)(32 + 64 + 16 + 16 + 4 + kNumStats + 2 + 2) * 4;
  static_assert((size_t)4 * kVocabSlots * NR * 4 <= kZBuf, "partial sums in a row buffer");
  static_assert(smem <= 160 * 1024, "LDS");
};

// Words of 8 bytes that a group exchanges, and where each kind begins: all ones at first | zeros at first
struct VocabLayout {
  size_t keys, bn, h, ones, p, zeros;
};
__host__ __device__ inline VocabLayout vocab_layout(int H, int nparts, int NS, int qmax) {
  const size_t quads = (size_t)NS * qmax;
  VocabLayout l;
  l.keys = quads * H;                          // z: [quad][H / 4][4 rows] four columns
  l.bn = l.keys + quads * nparts * 4;          // keys: [quad][part][4 rows]
  l.h = l.bn + quads * H;                      // bn: [quad][H / 4][4 rows] (part of the blank logit, of the squared norm)
  l.ones = l.h + (size_t)NS * H;               // h: [2][slot][H] words of 4 bytes
  l.p = kVocabSlots;                           // dec: [slot]
  l.zeros = l.p + (size_t)NS * H;              // p: [slot][H]
  return l;
}

// 16 bytes past the CU's cache (sc1), as an agent-scope load has it; the two words of 8 bytes may be of different times.
__device__ __forceinline__ u32x4 vocab_ld16(__amdgpu_buffer_rsrc_t r, int off) {
  return __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 16 | (int)0x80000000));
}
__device__ __forceinline__ __amdgpu_buffer_rsrc_t vocab_rsrc(const void *p, size_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, (int)bytes, 0x00020000);
}

// A slot before an iteration, in LDS: wave 4 moves all slots on from one iteration to the next.
struct __attribute__((aligned(16))) VocabSlot {
  int b, t, len, nwin;        // utterance, frame, length (t = len = 0: no utterance or done), frames of the window
  int sym, cnt;               // labels on the frame, labels so far
  int quads;                  // quads that the window may have | tags of the quads' next uses << 8
  int steps;                  // LSTM steps taken
};

// Waits for words that other waves of the workgroup write to LDS.  False: gave up (they always write them, at last because a wait of theirs has)
template <class Ask>
__device__ __forceinline__ bool vocab_wait(unsigned limit, const Ask &ask) {
  for (unsigned spins = 0; !__all(ask());)
    if (++spins > limit + (1u << 16)) return false;
  return true;
}

// recheck_row for the keys of up to 128 parts of 32 labels, two of each part: every label at or above `thresh`, and all labels of a part whose second key
// is, in fp32 (weight rows in bf16 times relu(e + p), four at a time); ties to the lowest label, blank the highest.  p lies in LDS.
template <int KS>
__device__ __forceinline__ int vocab_recheck(const ModelDev &m, const float *er, const float *p, float vblank, float thresh, float4 kA, float4 kB) {
  const int lane = threadIdx.x & 63, V = m.V;
  const bf16_t *w = reinterpret_cast<const bf16_t *>(m.w_out);
  float2 e[KS];
#pragma unroll
  for (int i = 0; i < KS; ++i) e[i] = *reinterpret_cast<const float2 *>(er + 2 * lane + 128 * i);
  float bestv = vblank;
  int besti = V, mycol = 0, nc = 0;   // lane i: the i-th candidate
  auto evaluate = [&]() {
    for (int c0 = 0; c0 < nc; c0 += 4) {
      int col[4];
      uint32_t x[4][KS];
      float o[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        col[k] = __builtin_amdgcn_readlane(mycol, min(c0 + k, nc - 1));
        o[k] = m.b_out[col[k]];
#pragma unroll
        for (int i = 0; i < KS; ++i) x[k][i] = *reinterpret_cast<const uint32_t *>(w + (size_t)col[k] * (128 * KS) + 2 * lane + 128 * i);
      }
      float a[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int i = 0; i < KS; ++i) {
        const float2 q = *reinterpret_cast<const float2 *>(p + 2 * lane + 128 * i);
        const float zx = fmaxf(e[i].x + q.x, 0.f), zy = fmaxf(e[i].y + q.y, 0.f);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          a[k] = fmaf(__uint_as_float(x[k][i] << 16), zx, a[k]);
          a[k] = fmaf(__uint_as_float(x[k][i] & 0xFFFF0000u), zy, a[k]);
        }
      }
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const float v = wave_sum(a[k]) + o[k];
        if (v > bestv || (v == bestv && col[k] < besti)) { bestv = v; besti = col[k]; }
      }
    }
    nc = 0;
  };
  auto add = [&](int col) {
    if (lane == nc) mycol = col;
    if (++nc == 64) evaluate();
  };
  for (int half = 0; half < 2; ++half) {
    const float k1 = half ? kB.x : kA.x, k2 = half ? kB.y : kA.y;
    unsigned long long whole = __ballot(key_val(k2) >= thresh), one = __ballot(key_val(k1) >= thresh && !(key_val(k2) >= thresh));
    for (; one; one &= one - 1) {
      const int src = __ffsll((long long)one) - 1;
      add((64 * half + src) * 32 + key_col(readlane_f32(k1, src)));
    }
    for (; whole; whole &= whole - 1) {
      const int c0 = (64 * half + __ffsll((long long)whole) - 1) * 32;
      for (int i = 0; i < 32 && c0 + i < V; ++i) add(c0 + i);
    }
  }
  evaluate();
  return besti;
}

template <int KS, int ROLE>
__device__ __forceinline__ void vocab_loop(const ModelDev &m, const CallDev &c, const GroupDev &gd, unsigned char *smem, int grp, int g) {
  using Cfg = VocabCfg<KS>;
  constexpr int H = Cfg::H, NR = Cfg::NR, QK = Cfg::QK, PPW = Cfg::PPW, UPW = Cfg::UPW, NC = Cfg::NC, ZST = Cfg::ZST;
  constexpr int kItems = (kVocabSlots * UPW + 511) / 512;
  bf16_t *zbuf = reinterpret_cast<bf16_t *>(smem + Cfg::oZ);
  float *recp = reinterpret_cast<float *>(smem + Cfg::oZ), *ering = reinterpret_cast<float *>(smem + Cfg::oE);
  float *predp = reinterpret_cast<float *>(smem + Cfg::oPred), *pst = reinterpret_cast<float *>(smem + Cfg::oP);
  float *recs = reinterpret_cast<float *>(smem + Cfg::oRec), *cst = reinterpret_cast<float *>(smem + Cfg::oC);
  float *pfull = reinterpret_cast<float *>(smem + Cfg::oPf), *bias = reinterpret_cast<float *>(smem + Cfg::oB);
  float *wbl = reinterpret_cast<float *>(smem + Cfg::oWb), *bpl = wbl + PPW;
  VocabSlot *slots = reinterpret_cast<VocabSlot *>(smem + Cfg::oS);
  int *qtab = reinterpret_cast<int *>(smem + Cfg::oQ), *info = reinterpret_cast<int *>(smem + Cfg::oI), *emaps = info + 32;
  volatile int *stat = emaps + 64;
  int *rech = emaps + 80, *head = rech + 16, *counts = head + 4, *fail = counts + kNumStats + 2, *near_w = fail + 1;

  int lane = threadIdx.x & 63, tid = threadIdx.x, tid1 = tid & 255, l15 = lane & 15, l4 = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), w4 = wave & 3;
  const int V = m.V, NS = gd.NS, nparts = c.nparts_tiny, ring = gd.ring, rlog = 31 - __clz(ring), qmax = gd.qmax;
  unsigned *abort_word = gd.bar + grp * kGroupBarInts;
  const VocabLayout lay = vocab_layout(H, nparts, NS, qmax);
  unsigned long long *ones = gd.vx + (size_t)grp * lay.ones, *zeros = gd.v0 + (size_t)grp * lay.zeros;
  unsigned long long *kx = ones + lay.keys, *bx = ones + lay.bn, *dx = zeros, *px = zeros + lay.p;
  unsigned *hx = reinterpret_cast<unsigned *>(ones + lay.h);
  const int unit0 = g * UPW, col0 = g * PPW;

  // ---- weights into registers
  f16x8 wo[ROLE == 0 ? 8 * KS : 1];                                          // 32 columns of W_out over the whole of K, scaled
  bf16x8 wr[ROLE == 1 ? Cfg::LT : 1][KS], wp[ROLE == 1 ? Cfg::PT : 1][KS];   // a quarter of K of the recurrent rows and of the projection rows
  const int part = 32 * w4 + g;                                              // ROLE 0
  if constexpr (ROLE == 0) {
    const int col = min(part * 32 + (lane & 31), m.Vpad - 1);
    const bf16_t *src = reinterpret_cast<const bf16_t *>(m.w_out) + (size_t)col * H + (lane >> 5) * 8;
#pragma unroll
    for (int i = 0; i < 8 * KS; ++i) {
      const u32x4 b = *reinterpret_cast<const u32x4 *>(src + i * 16);
      u32x4 h;
#pragma unroll
      for (int q = 0; q < 4; ++q) h[q] = pack_f16x2(__uint_as_float(b[q] << 16) * m.w16_scale, __uint_as_float(b[q] & 0xFFFF0000u) * m.w16_scale);
      wo[i] = __builtin_bit_cast(f16x8, h);
    }
  } else {
#pragma unroll
    for (int t = 0; t < Cfg::LT; ++t) {
      const bf16_t *src = reinterpret_cast<const bf16_t *>(m.w_cat[0]) + (size_t)(unit0 * 4 + 16 * t + l15) * H + w4 * QK + l4 * 8;
#pragma unroll
      for (int i = 0; i < KS; ++i) wr[t][i] = *reinterpret_cast<const bf16x8 *>(src + i * 32);
    }
#pragma unroll
    for (int t = 0; t < Cfg::PT; ++t) {
      const bf16_t *src = reinterpret_cast<const bf16_t *>(m.w_pred) + (size_t)(col0 + min(16 * t + l15, PPW - 1)) * H + w4 * QK + l4 * 8;
#pragma unroll
      for (int i = 0; i < KS; ++i) wp[t][i] = *reinterpret_cast<const bf16x8 *>(src + i * 32);
    }
  }
  // ---- state after the start token, constants
  for (int i = tid; i < NS * NR; i += 512) recs[i] = m.start_rec[unit0 * 4 + i % NR];
  for (int i = tid; i < NS * UPW; i += 512) cst[i] = m.start_c[unit0 + i % UPW];
  for (int i = tid; i < NS * PPW; i += 512) pst[i] = m.start_p[col0 + i % PPW];
  for (int i = tid; i < H; i += 512) pfull[i] = m.start_p[i];
  for (int i = tid; i < 128; i += 512) {
    const int col = (32 * (i >> 5) + g) * 32 + (i & 31);
    bias[i] = col < V ? m.b_out[col] : kKeyNone;   // what is added to kKeyNone vanishes in it
  }
  for (int i = tid; i < PPW; i += 512) {
    wbl[i] = m.w_blank[col0 + i];
    bpl[i] = m.b_pred[col0 + i];
  }
  for (int i = tid; i < kNumStats + 2; i += 512) counts[i] = 0;
  if (tid < 16) stat[tid] = 0;
  if (tid == 0) *fail = 0;
  // ---- every slot's utterance: dealt by falling length, one to every group in turn
  if (wave == 4) {
    const int n_order = *gd.n_order, rank = lane * gd.NG + grp;
    VocabSlot s{};
    if (lane < NS && rank < n_order) {
      s.b = gd.order[rank];
      s.len = c.len[s.b];
      s.nwin = min(min(gd.reach, 4), s.len);
    }
    s.quads = 1;
    if (lane < 32) slots[lane] = s;
    const unsigned long long act = __ballot(s.nwin > 0);
    if (lane == 0) { head[0] = (int)(unsigned)act; head[1] = 0; }
  }
  group_barrier();

  // The frames that the slots have come to need since frame t0 (of `before`; null: all), this workgroup's columns, into their rings: lane =
  // (slot, place in its ring)
  auto load_frames = [&](const VocabSlot *before, const VocabSlot *now) {
    const int s = tid >> rlog, pos = tid & (ring - 1), b = now[s].b, len = now[s].len, t = now[s].t;
    const int from = before ? min(len, before[s].t + ring) : 0, f = from + ((pos - from) & (ring - 1));
    const unsigned lds = (unsigned)(unsigned long long)(__attribute__((address_space(3))) const float *)ering + (unsigned)wave * 1024u;
    if (f < min(len, t + ring)) {
      const float *src = c.e + (size_t)((unsigned)b * (unsigned)c.T + (unsigned)f) * H + col0;
#pragma unroll
      for (int i = 0; i < NC; ++i) group_load_lds(src + 4 * i, lds + (unsigned)i * 8192u);
    }
  };
  // The next iteration's quads, in the order of their slots (one wave; em: slots with a new projection)
  auto list_quads = [&](const VocabSlot *now, unsigned em) {
    const int t = now[lane & 31].t, nwin = lane < 32 ? now[lane & 31].nwin : 0, tags = now[lane & 31].quads >> 8, nqe = (nwin + 3) >> 2;
    const unsigned long long m1 = __ballot(nqe >= 1), m2 = __ballot(nqe >= 2), m3 = __ballot(nqe >= 3), m4 = __ballot(nqe >= 4), below = (1ull << lane) - 1ull;
    const int at = __popcll(m1 & below) + __popcll(m2 & below) + __popcll(m3 & below) + __popcll(m4 & below);
    const int rank = lane < 32 && (em >> lane) & 1 ? __popc(em & (unsigned)below) : 63;
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (q < nqe) qtab[at + q] = lane | q << 5 | ((tags >> q) & 1) << 7 | ((t + 4 * q) & (ring - 1)) << 8 | min(4, nwin - 4 * q) << 16 | rank << 20;
    if (lane == 0) head[2] = __popcll(m1) + __popcll(m2) + __popcll(m3) + __popcll(m4);
  };
  load_frames(nullptr, slots);
  if (wave == 1) list_quads(slots, 0u);
  // ---- where the workgroups sit: XCD numbers, exchanged with device-wide stores
  if (wave == 0) {
    unsigned xcc;
    asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(xcc));
    xcc = (xcc & 15u) + 1u;
    unsigned *bw = abort_word + 64;
    if (lane == 0) __hip_atomic_store(bw + g * 32, xcc, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    unsigned v = xcc;
    const bool got = group_poll(abort_word, gd.start_limit, [&]() {
      if (lane < 32) v = __hip_atomic_load(bw + lane * 32, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      return v != 0u;
    });
    const bool same = __all(v == xcc);
    if (lane == 0) {
      *near_w = same ? 1 : 0;
      if (!got) *fail = 1;
      if (g == 0) abort_word[1] = same ? 2u : 1u;
    }
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  group_barrier();
  const bool near = __builtin_amdgcn_readfirstlane(*near_w);
  if (*fail) return;
  const __amdgpu_buffer_rsrc_t zr = vocab_rsrc(ones, lay.keys * 8), hr = vocab_rsrc(hx, (size_t)2 * NS * H * 4);

  // The hidden vectors of 16 slots with a label (of the list emap) as operand rows: lane (row l15, K group l4) its 8 units per step of 32 of this wave's
  // quarter of K, as bf16 hi and lo
  bf16x8 hi[ROLE == 1 ? KS : 1], lo[ROLE == 1 ? KS : 1];
  auto hidden_rows = [&](const int *emap, int tile, int n_em) -> bool {
    const int en = emap[min(16 * tile + l15, n_em - 1)];
    const unsigned tag = (unsigned)((en >> 9) & 1) << 14;
    const int base = ((((en >> 8) & 1) * NS + (en & 255)) * H + w4 * QK + l4 * 8) * 4;
    u32x4 x[KS][2];
    const bool got = group_poll(abort_word, gd.spin_limit, [&]() {
      asm volatile("" ::: "memory");
      unsigned wrong = 0;
#pragma unroll
      for (int i = 0; i < KS; ++i)
#pragma unroll
        for (int h = 0; h < 2; ++h) x[i][h] = vocab_ld16(hr, base + i * 128 + h * 16);
#pragma unroll
      for (int i = 0; i < KS; ++i)
#pragma unroll
        for (int h = 0; h < 2; ++h) wrong |= (x[i][h][0] ^ tag) | (x[i][h][1] ^ tag) | (x[i][h][2] ^ tag) | (x[i][h][3] ^ tag);
      return (wrong & 0x4000u) == 0u;
    });
#pragma unroll
    for (int i = 0; i < KS; ++i) {
      u32x4 a, r;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const unsigned y0 = x[i][q >> 1][2 * (q & 1)], y1 = x[i][q >> 1][2 * (q & 1) + 1];
        a[q] = __builtin_amdgcn_perm(y1, y0, 0x05040100u) & 0xBFFFBFFFu;
        r[q] = __builtin_amdgcn_perm(y1, y0, 0x07060302u);
      }
      hi[i] = __builtin_bit_cast(bf16x8, a);
      lo[i] = __builtin_bit_cast(bf16x8, r);
    }
    return got;
  };
  f32x4 racc[ROLE == 1 ? Cfg::LT : 1];   // recurrent sums of the step after the last label, this wave's quarter of K, for the last tile of slots
  auto recurrent_sums = [&]() {
#pragma unroll
    for (int t = 0; t < Cfg::LT; ++t) racc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < KS; ++i)
#pragma unroll
      for (int t = 0; t < Cfg::LT; ++t) {
        racc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(hi[i], wr[t][i], racc[t], 0, 0, 0);
        racc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(lo[i], wr[t][i], racc[t], 0, 0, 0);
      }
  };

  const float unscale = 1.f / m.w16_scale;   // a power of two
  bool bad = false;   // a wait of this wave has given up: told to the workgroup ahead of the decisions' barrier
  for (int it = 0;; ++it) {
    // opaque: see wind_group_kernel
    asm volatile("" : "+v"(lane), "+v"(tid), "+v"(tid1));
    l15 = lane & 15;
    l4 = lane >> 4;
    const unsigned act = (unsigned)__builtin_amdgcn_readfirstlane(head[0]), em = (unsigned)__builtin_amdgcn_readfirstlane(head[1]);
    const int nquads = __builtin_amdgcn_readfirstlane(head[2]), n_em = __popc(em), nch = (nquads + 7) >> 3;
    VocabSlot *now = slots + (it & 1) * kVocabSlots, *next = slots + ((it & 1) ^ 1) * kVocabSlots;
    const int *emap = emaps + 32 * vocab_emit_list(it);
    int *emap_next = emaps + 32 * vocab_emit_list(it + 1);
    const unsigned stamp = (unsigned)it + 1u;
    if (!act) break;
    if constexpr (ROLE == 0) {
      // ---- this workgroup's columns of the window rows: item (quad, 4 columns, row).  The four partial sums of a new projection lie with
      // the four rows' threads
      for (int x0 = 0; x0 < 4 * NC * nquads; x0 += 256) {
        const int x = (x0 + tid1) >> 2, r = tid1 & 3, qi = x / NC, i = x - qi * NC;
        if (qi >= nquads) break;
        const int q = qtab[qi], s = q & 31, qq = (q >> 5) & 3, pos = (((q >> 8) & 31) + r) & (ring - 1), rank = (q >> 20) & 63;
        const unsigned tag = (unsigned)(q >> 7) & 1u, tagz = tag ? 0x80008000u : 0u;
        const bool valid = r < ((q >> 16) & 7), fresh = rank < 63;
        f32x4 p = *reinterpret_cast<const f32x4 *>((fresh ? predp + (r * kVocabSlots + rank) * PPW : pst + s * PPW) + 4 * i);
        const f32x4 e = *reinterpret_cast<const f32x4 *>(ering + (size_t)(i * 512 + s * ring + pos) * 4);
        const f32x4 b4 = *reinterpret_cast<const f32x4 *>(bpl + 4 * i), w = *reinterpret_cast<const f32x4 *>(wbl + 4 * i);
        float y[4], nrm = 0.f;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          float v = fresh || r == 0 ? p[k] : 0.f;
          v += dpp_f32<kDppQuadXor1>(v);
          v += dpp_f32<kDppQuadXor2>(v);
          if (fresh) v += b4[k];
          p[k] = v;
          y[k] = valid ? fmaxf(e[k] + v, 0.f) : 0.f;
          nrm = fmaf(y[k], y[k], nrm);
        }
        nrm = fmaxf(fmaxf(y[0], y[1]), fmaxf(y[2], y[3])) == INFINITY ? 3.f * kNormInfinite : fminf(nrm, kNormPart);
        const float dot = fmaf(y[3], w[3], fmaf(y[2], w[2], fmaf(y[1], w[1], y[0] * w[0])));
        const int quad = s * qmax + qq;
        group_st(ones + (size_t)(quad * H + (g * NC + i) * 4 + r), (pack_f16x2(y[0], y[1]) & 0x7FFF7FFFu) | tagz,
                 (pack_f16x2(y[2], y[3]) & 0x7FFF7FFFu) | tagz, near);
        group_st(bx + (size_t)(quad * H + (g * NC + i) * 4 + r), __float_as_uint(dot), (__float_as_uint(nrm) & ~1u) | tag, near);
        if (fresh && qq == 0) {
          const float mine = r == 0 ? p[0] : r == 1 ? p[1] : r == 2 ? p[2] : p[3];
          pst[s * PPW + 4 * i + r] = mine;
          group_st(px + (size_t)(s * H + col0 + 4 * i + r), __float_as_uint(mine), stamp, near);
        }
      }
    } else {
      if (n_em) recurrent_sums();   // beside that: of the next step, for the tile of hidden vectors at hand
    }
    // ---- chunks of 8 quads: waves 4-7 fetch the next, waves 0-3 multiply the last
    for (int ch = 0; ch <= nch; ++ch) {
      if constexpr (ROLE == 1) {
        if (ch < nch) {
          bf16_t *dst = zbuf + (ch & 1) * (Cfg::kZBuf / 2) + 8 * w4 * ZST;
          const int q0 = ch * 8 + 2 * w4;
          int src[2];
          unsigned tag[2];
#pragma unroll
          for (int k = 0; k < 2; ++k) {
            const int q = __builtin_amdgcn_readfirstlane(qtab[min(q0 + k, nquads - 1)]);
            src[k] = ((q & 31) * qmax + ((q >> 5) & 3)) * (H * 8) + lane * 16;
            tag[k] = (q >> 7) & 1 ? 0x80008000u : 0u;
          }
          if (q0 < nquads) {
            u32x4 x[2][KS];
            const bool got = group_poll(abort_word, gd.spin_limit, [&]() {
              asm volatile("" ::: "memory");
#pragma unroll
              for (int k = 0; k < 2; ++k)
#pragma unroll
                for (int i = 0; i < KS; ++i) x[k][i] = vocab_ld16(zr, src[k] + i * 1024);
              unsigned wrong = 0;
#pragma unroll
              for (int k = 0; k < 2; ++k)
#pragma unroll
                for (int i = 0; i < KS; ++i) wrong |= (x[k][i][0] ^ tag[k]) | (x[k][i][1] ^ tag[k]) | (x[k][i][2] ^ tag[k]) | (x[k][i][3] ^ tag[k]);
              return (wrong & 0x80008000u) == 0u;
            });
            bad |= !got;
#pragma unroll
            for (int k = 0; k < 2; ++k)
#pragma unroll
              for (int i = 0; i < KS; ++i) {
                // pair lane + 64 i of the quad: columns 4 (pair / 2) .., rows 2 (pair & 1) and the next
                bf16_t *d = dst + (4 * k + 2 * (lane & 1)) * ZST + 4 * (lane >> 1) + 128 * i;
                *reinterpret_cast<u32x2 *>(d) = u32x2{x[k][i][0] & 0x7FFF7FFFu, x[k][i][1] & 0x7FFF7FFFu};
                *reinterpret_cast<u32x2 *>(d + ZST) = u32x2{x[k][i][2] & 0x7FFF7FFFu, x[k][i][3] & 0x7FFF7FFFu};
              }
          }
        } else if (g < NS && ((em >> g) & 1)) {   // this workgroup's own slot has a new projection: for near-ties
          unsigned long long u[(QK + 63) / 64];
          const bool got = group_poll(abort_word, gd.spin_limit, [&]() {
            bool ok = true;
#pragma unroll
            for (int k = 0; k < (QK + 63) / 64; ++k) u[k] = group_ld(px + (size_t)g * H + w4 * QK + min(lane + 64 * k, QK - 1));
#pragma unroll
            for (int k = 0; k < (QK + 63) / 64; ++k) ok = ok && (unsigned)(u[k] >> 32) == stamp;
            return ok;
          });
          bad |= !got;
#pragma unroll
          for (int k = 0; k < (QK + 63) / 64; ++k)
            if (lane + 64 * k < QK) pfull[w4 * QK + lane + 64 * k] = __uint_as_float((unsigned)u[k]);
        }
      } else if (ch > 0 && part < nparts) {
        const bf16_t *zs = zbuf + ((ch - 1) & 1) * (Cfg::kZBuf / 2) + (lane & 31) * ZST + (lane >> 5) * 8;
        f32x16 acc;
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[r] = 0.f;
        // the rows' operands are read three steps of two ahead
        f16x8 zf[4][2];
        auto read_rows = [&](int s) {
#pragma unroll
          for (int i = 0; i < 2; ++i) zf[s & 3][i] = *reinterpret_cast<const f16x8 *>(zs + (2 * s + i) * 16);
        };
#pragma unroll
        for (int s = 0; s < 3; ++s) read_rows(s);
#pragma unroll
        for (int s = 0; s < 4 * KS; ++s) {
          if (s + 3 < 4 * KS) read_rows(s + 3);
#pragma unroll
          for (int i = 0; i < 2; ++i) acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(wo[2 * s + i], zf[s & 3][i], acc, 0, 0, 0);
          __builtin_amdgcn_sched_barrier(0);   // keeps the reads there: registers
        }
        // accumulator r: column 8 (r / 4) + 4 (lane / 32) + r % 4 of the part; row lane % 32
        float k1 = kKeyNone, k2 = kKeyNone;
        const int hi4 = 4 * (lane >> 5);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const f32x4 b4 = *reinterpret_cast<const f32x4 *>(bias + 32 * w4 + 8 * r + hi4);
#pragma unroll
          for (int k = 0; k < 4; ++k) push_top2(k1, k2, make_key(fmaf(acc[4 * r + k], unscale, b4[k]), 8 * r + k + hi4));
        }
        merge_top2(k1, k2, xor32_f32(k1), xor32_f32(k2));
        const int qi = (ch - 1) * 8 + ((lane & 31) >> 2);
        if (lane < 32 && qi < nquads) {
          const int q = qtab[qi], quad = (q & 31) * qmax + ((q >> 5) & 3);
          group_st(kx + ((size_t)quad * nparts + part) * 4 + (lane & 3), __float_as_uint(k1), __float_as_uint(key_with_tag(k2, (q >> 7) & 1)), near);
        }
      }
      group_barrier();
    }
    if constexpr (ROLE == 1) {
      // ---- the recurrent sums that the last labels left behind
      for (int tile = (n_em - 1) >> 4; n_em > 0 && tile >= 0; --tile) {
        if (16 * tile + 16 < n_em) {   // not the tile whose sums are at hand
          bad |= !hidden_rows(emap, tile, n_em);
          recurrent_sums();
        }
#pragma unroll
        for (int t = 0; t < Cfg::LT; ++t)
#pragma unroll
          for (int r = 0; r < 4; ++r) recp[(w4 * kVocabSlots + 16 * tile + 4 * l4 + r) * NR + 16 * t + l15] = racc[t][r];
      }
    } else {
      // ---- the decision of this workgroup's own slot
      if (g < NS && (act >> (g & 31)) & 1) {
        const int n = __builtin_amdgcn_readfirstlane(now[g].nwin), tags = __builtin_amdgcn_readfirstlane(now[g].quads) >> 8,
                  b = __builtin_amdgcn_readfirstlane(now[g].b), t = __builtin_amdgcn_readfirstlane(now[g].t), nq = (n + 3) >> 2;
        const int mark = ((it + 1) & 0x1FFFF) << 14;   // tells this iteration's words in LDS from the last one's
        auto first = [](unsigned long long u) { return __uint_as_float((unsigned)u); };
        auto second = [](unsigned long long u) { return __uint_as_float((unsigned)(u >> 32)); };
        // The first of the window's rows before `rows` that is not blank (-1: none), once that is settled
        auto settled = [&](int rows, int &st) -> int {
          int at = -1;
          bad |= !vocab_wait(gd.spin_limit, [&]() {
            st = lane < rows ? stat[lane & 15] : mark | V;
            const unsigned long long nb = __ballot((st & kTie) != V);
            at = nb ? __ffsll((long long)nb) - 1 : -1;
            return (st & ~kTie) == mark && (at < 0 || (__builtin_amdgcn_readlane(st, max(at, 0)) & kTie) != kTie);
          });
          return at;
        };
        // A row that fp16 cannot hold: the groups give the call up, and this wave's rows are blank so that nobody here waits for them
        auto leave = [&]() {
          bad = true;
          if (lane == 0) __hip_atomic_store(abort_word, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        };
        if (nq == 1) {
          // one quad: row w4, lane with the keys of parts lane and lane + 64
          const unsigned long long *kr = kx + (size_t)g * qmax * nparts * 4 + w4, *br = bx + (size_t)g * qmax * H + w4;
          const int tag = tags & 1;
          constexpr int kBn = (H / 4 + 63) / 64;
          unsigned long long ua, ub, v[kBn];
          bad |= !group_poll(abort_word, gd.spin_limit, [&]() {
            ua = lane < nparts ? group_ld(kr + 4 * lane) : 0ull;
            ub = lane + 64 < nparts ? group_ld(kr + 4 * (lane + 64)) : 0ull;
#pragma unroll
            for (int k = 0; k < kBn; ++k) v[k] = lane + 64 * k < H / 4 ? group_ld(br + 4 * (lane + 64 * k)) : 0ull;
            bool ok = (lane >= nparts || key_tag(second(ua)) == tag) && (lane + 64 >= nparts || key_tag(second(ub)) == tag);
#pragma unroll
            for (int k = 0; k < kBn; ++k) ok = ok && (lane + 64 * k >= H / 4 || (int)((v[k] >> 32) & 1u) == tag);
            return ok;
          });
          float4 kA = no_keys(), kB = no_keys();
          if (lane < nparts) { kA.x = first(ua); kA.y = key_with_tag(second(ua), 0); }
          if (lane + 64 < nparts) { kB.x = first(ub); kB.y = key_with_tag(second(ub), 0); }
          float dot = 0.f, nrm = 0.f;
#pragma unroll
          for (int k = 0; k < kBn; ++k) { dot += first(v[k]); nrm += second(v[k]); }
          const float vblank = wave_sum(dot) + m.b_out[V], norm2 = wave_sum(nrm);
          const float kbest = wave_max_f32(fmaxf(kA.x, kB.x)), vbest = key_val(kbest), top = fmaxf(vbest, vblank);
          const float thresh = top - vocab_band(m, sqrtf(norm2), top);
          int label = V;   // also of a row with an infinite unit
          if (w4 < n && norm2 > kZ16Max * kZ16Max && norm2 < kNormInfinite) {
            leave();
          } else if (w4 < n && norm2 < kNormInfinite && !(vbest < thresh)) {
            const int cnt = __popcll(__ballot(key_val(kA.x) >= thresh)) + __popcll(__ballot(key_val(kA.y) >= thresh)) +
                            __popcll(__ballot(key_val(kB.x) >= thresh)) + __popcll(__ballot(key_val(kB.y) >= thresh));
            if (cnt == 1 && vblank < thresh) {
              int col = 0;
              if (kA.x == kbest) col = lane * 32 + key_col(kbest);
              if (kB.x == kbest) col = (lane + 64) * 32 + key_col(kbest);
              label = min(wave_max_i32(col), V);
            } else {
              label = kTie;
            }
          }
          if (lane == 0) { rech[w4] = 0; stat[w4] = mark | label; }
          int st;
          if (label == kTie && settled(w4, st) < 0) {
            label = vocab_recheck<KS>(m, c.e + ((size_t)b * c.T + t + w4) * H, pfull, vblank, thresh, kA, kB);
            if (lane == 0) { rech[w4] = 1; stat[w4] = mark | label; }
          }
        } else if (w4 < nq) {
          // a wave per quad: 16 lanes per row, lane l15 with the keys of parts l15, l15 + 16, ..
          const unsigned long long *kr = kx + (size_t)(g * qmax + w4) * nparts * 4, *br = bx + (size_t)(g * qmax + w4) * H;
          const int tag = (tags >> w4) & 1;
          unsigned long long u[8], v[2 * KS];
          bad |= !group_poll(abort_word, gd.spin_limit, [&]() {
            bool ok = true;
#pragma unroll
            for (int k = 0; k < 8; ++k) u[k] = l15 + 16 * k < nparts ? group_ld(kr + 4 * (l15 + 16 * k) + l4) : 0ull;
#pragma unroll
            for (int k = 0; k < 2 * KS; ++k) v[k] = group_ld(br + 4 * (l15 + 16 * k) + l4);
#pragma unroll
            for (int k = 0; k < 8; ++k) ok = ok && (l15 + 16 * k >= nparts || key_tag(second(u[k])) == tag);
#pragma unroll
            for (int k = 0; k < 2 * KS; ++k) ok = ok && (int)((v[k] >> 32) & 1u) == tag;
            return ok;
          });
          float dot = 0.f, nrm = 0.f, kbest = kKeyNone;
#pragma unroll
          for (int k = 0; k < 2 * KS; ++k) { dot += first(v[k]); nrm += second(v[k]); }
#pragma unroll
          for (int k = 0; k < 8; ++k) kbest = fmaxf(kbest, l15 + 16 * k < nparts ? first(u[k]) : kKeyNone);
          kbest = row16_max_f32(kbest);
          const float vblank = row16_sum_f32(dot) + m.b_out[V], norm2 = row16_sum_f32(nrm), vbest = key_val(kbest), top = fmaxf(vbest, vblank);
          const float thresh = top - vocab_band(m, sqrtf(norm2), top);
          int cnt = 0, col = 0;   // with NaN logits no key is a label's
#pragma unroll
          for (int k = 0; k < 8; ++k)
            if (l15 + 16 * k < nparts) {
              cnt += (key_val(first(u[k])) >= thresh) + (key_val(key_with_tag(second(u[k]), 0)) >= thresh);
              if (first(u[k]) == kbest) col = (l15 + 16 * k) * 32 + key_col(kbest);
            }
          cnt = row16_sum_i32(cnt);
          col = row16_max_i32(col);
          const int j = 4 * w4 + l4;
          int label = V;
          if (j < n && norm2 < kNormInfinite && !(vbest < thresh)) label = cnt == 1 && vblank < thresh ? min(col, V) : kTie;
          if (__any(j < n && norm2 > kZ16Max * kZ16Max && norm2 < kNormInfinite)) {
            leave();
            label = V;
          }
          if (l15 == 0) { rech[j] = 0; stat[j] = mark | label; }
          // near-ties ahead of the first certain label, in the order of their rows
          for (unsigned long long todo = __ballot(l15 == 0 && label != V); todo; todo &= todo - 1) {
            const int src = __ffsll((long long)todo) - 1, row = 4 * w4 + (src >> 4);
            if (__builtin_amdgcn_readlane(label, src) != kTie) break;
            int st;
            if (settled(row, st) >= 0) break;
            float4 kA = no_keys(), kB = no_keys();
            const unsigned long long *kt = kr + (src >> 4);
            if (lane < nparts) { const unsigned long long x = group_ld(kt + 4 * lane); kA.x = first(x); kA.y = key_with_tag(second(x), 0); }
            if (lane + 64 < nparts) { const unsigned long long x = group_ld(kt + 4 * (lane + 64)); kB.x = first(x); kB.y = key_with_tag(second(x), 0); }
            const int l = vocab_recheck<KS>(m, c.e + ((size_t)b * c.T + t + row) * H, pfull, readlane_f32(vblank, src), readlane_f32(thresh, src), kA, kB);
            if (lane == 0) { rech[row] = 1; stat[row] = mark | l; }
            if (l != V) break;
          }
        }
        // ---- the slot's outcome goes to everybody: its first label and that label's row, if any.  Behind everybody's reads of the slot's words
        if (w4 == 0) {
          int st;
          const int at = settled(4 * nq, st), tok = at < 0 ? 0 : __builtin_amdgcn_readlane(st, max(at, 0)) & kTie;
          if (lane == 0) group_st(dx + g, (unsigned)(at + 1) << 16 | (unsigned)min(tok, V), stamp, near);
        }
      }
    }
    if (ROLE == 1 && wave == 4) {
      // ---- one wave moves the slots on: lane s has slot s
      VocabSlot s = now[lane & 31];
      const bool on = lane < 32 && (act >> lane) & 1;
      unsigned long long u = 0;
      bad |= !group_poll(abort_word, gd.spin_limit, [&]() {
        if (on) u = group_ld(dx + lane);
        return !on || (unsigned)(u >> 32) == stamp;
      });
      const int first = (int)((unsigned)u >> 16) - 1, tok = (int)(u & 0xFFFFu);
      bool emits = false;
      if (on) {
        const WindowOutcome wo = window_outcome(c, make_int4(s.b, s.t, s.len, s.sym), s.cnt, s.nwin, first, tok, V, 0, false);
        const int nqe = (s.nwin + 3) >> 2;
        s.t = wo.slot.y; s.sym = wo.slot.w; s.cnt = wo.cnt;
        s.quads = (first < 0 ? min(2 * (s.quads & 255), qmax) : 1) | ((s.quads >> 8) ^ ((1 << nqe) - 1)) << 8;
        emits = (wo.flag & 2) != 0;
        if (emits) ++s.steps;
        if (!(wo.flag & 1)) s.t = s.len = 0;
        s.nwin = min(min(gd.reach, 4 * (s.quads & 255)), s.len - s.t);
      }
      const unsigned em1 = (unsigned)__ballot(emits), act1 = (unsigned)__ballot(lane < 32 && s.nwin > 0), below = (1u << (lane & 31)) - 1u;
      if (lane < 32) {
        next[lane] = s;
        info[lane] = (emits ? 1 << 15 | tok : 0) | ((em >> lane) & 1 ? __popc(em & below) : 63) << 16 | ((s.steps - 1) & 3) << 24;
        if (emits) emap_next[__popc(em1 & below)] = lane | ((s.steps - 1) & 3) << 8;
        if (lane == g) { head[3] = (int)(unsigned)u; }
      }
      if (lane == 0) { head[0] = (int)act1; head[1] = (int)em1; }
    }
    if (bad && lane == 0) *fail = 1;
    group_barrier();
    if (*fail) return;
    load_frames(now, next);
    // ---- LSTM step: item (slot, unit of this workgroup's); first what the last step's products left behind
    {
      f32x4 x[kItems], rv[kItems];
      int in[kItems];
#pragma unroll
      for (int k = 0; k < kItems; ++k) {
        const int i = tid + 512 * k, s = i / UPW, u = i - s * UPW;
        in[k] = s < NS ? info[s] : 63 << 16;
        x[k] = f32x4{0.f, 0.f, 0.f, 0.f};
        if ((in[k] >> 15) & 1) x[k] = *reinterpret_cast<const f32x4 *>(m.emb_gates + (unsigned)(in[k] & 0x7FFF) * (4u * H) + (unsigned)((unit0 + u) * 4));   // fits 32 bits: checked by the host
      }
#pragma unroll
      for (int k = 0; k < kItems; ++k) {
        const int i = tid + 512 * k, rank = (in[k] >> 16) & 63;
        rv[k] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (i < NS * UPW) {
          if (rank < 63) {
            const f32x4 *rp = reinterpret_cast<const f32x4 *>(recp + rank * NR + 4 * (i % UPW));
            rv[k] = (rp[0] + rp[kVocabSlots * UPW]) + (rp[2 * kVocabSlots * UPW] + rp[3 * kVocabSlots * UPW]);
            *reinterpret_cast<f32x4 *>(recs + 4 * i) = rv[k];
          } else rv[k] = *reinterpret_cast<const f32x4 *>(recs + 4 * i);
        }
      }
#pragma unroll
      for (int k = 0; k < kItems; ++k) {
        const int i = tid + 512 * k, s = i / UPW, u = i - s * UPW;
        if (!((in[k] >> 15) & 1)) continue;
        const f32x4 pre = rv[k] + x[k];
        const float ig = 1.f / (1.f + expf(-pre[0])), fg = 1.f / (1.f + expf(-pre[1])), gg = tanhf(pre[2]), og = 1.f / (1.f + expf(-pre[3]));
        const float cn = fg * cst[i] + ig * gg, hv = og * tanhf(cn);
        cst[i] = cn;
        const unsigned hb = f32_to_bf16_bits(hv), lb = f32_to_bf16_bits(hv - bf16_bits_to_f32(hb));
        // |h| <= 1: bit 14 is free for the tag.  A value that is not a number goes into the lower half
        const unsigned word = fabsf(hv) <= 1.f ? hb | lb << 16 : 0x7FC00000u;
        group_publish(hx + (size_t)(((in[k] >> 24) & 1) * NS + s) * H + unit0 + u, (word & ~0x4000u) | (unsigned)((in[k] >> 25) & 1) << 14, near);
      }
    }
    if constexpr (ROLE == 1) {
      // ---- the projection columns of the new hidden vectors: partial sums over this wave's quarter of K
      const int n_new = __popc((unsigned)__builtin_amdgcn_readfirstlane(head[1]));
      for (int tile = 0; 16 * tile < n_new; ++tile) {
        bad |= !hidden_rows(emap_next, tile, n_new);
#pragma unroll
        for (int t = 0; t < Cfg::PT; ++t) {
          f32x4 a = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int i = 0; i < KS; ++i) {
            a = __builtin_amdgcn_mfma_f32_16x16x32_bf16(hi[i], wp[t][i], a, 0, 0, 0);
            a = __builtin_amdgcn_mfma_f32_16x16x32_bf16(lo[i], wp[t][i], a, 0, 0, 0);
          }
          if (16 * t + l15 < PPW)
#pragma unroll
            for (int r = 0; r < 4; ++r) predp[(w4 * kVocabSlots + 16 * tile + 4 * l4 + r) * PPW + 16 * t + l15] = a[r];
        }
      }
    } else if (wave == 0) {
      list_quads(next, (unsigned)__builtin_amdgcn_readfirstlane(head[1]));
      // Rows past the first quad may go without a decision for any time: their words' marks, 17 bits of the iteration, must not come round again
      if (((it + 2) & 0xFFFF) == 0 && lane < 16) stat[lane] = ((it + 1) & 0x1FFFF) << 14;
    } else if (wave == 1 && g < NS && (act >> (g & 31)) & 1) {
      // ---- the slot's outputs and the call's counters, in windows of the caller's size (as in group_outcome; one function for both makes decodes of the smallest
      // fp32 models 1 to 2 % slower: 66.0 -> 66.7 us, 91.8 -> 93.5)
      const unsigned long long again = __ballot(lane < 16 && lane < now[g].nwin && rech[lane & 15] != 0);
      if (lane == 0) {
        const VocabSlot s = now[g];
        const int first = (int)((unsigned)head[3] >> 16) - 1, tok = head[3] & 0xFFFF;
        const WindowOutcome wo = window_outcome(c, make_int4(s.b, s.t, s.len, s.sym), s.cnt, s.nwin, first, tok, V, 0, true);
        int *open = counts + kNumStats;
        const int ph = open[1], seen = ph + (first < 0 ? s.nwin : first), full = (int)(((unsigned)seen * gd.win_inv) >> 16), rem = seen - full * gd.win;
        const bool closes = first >= 0 || (rem > 0 && s.t + s.nwin == s.len);
        const int n_last = first < 0 ? rem : min(gd.win, s.len - (s.t + first - rem)), blanks = full * gd.win;
        const int forced = (int)((wo.ev >> 29) & 1u), looked = first < 0 ? 16 : min(16, (full + 1) * gd.win - ph);
        open[0] += full + closes;
        open[1] = closes ? 0 : rem;
        counts[ST_ITER] = open[0];
        counts[ST_WINDOWS] += full + closes;
        counts[ST_ROWS] += blanks + (closes ? n_last : 0);
        counts[ST_USEFUL] += blanks + (first >= 0 ? rem + 1 : closes ? rem : 0);
        counts[ST_RECHECK] += __popc((unsigned)again & ((1u << looked) - 1u));
        counts[ST_LABELS] += (int)((wo.ev >> 28) & 1u);
        counts[ST_FORCED] += forced;
        counts[ST_OVERFLOW] += (int)((wo.ev >> 30) & 1u);
        counts[kStatJump0 + gd.win] += full;
        if (closes) ++counts[kStatJump0 + rem + forced];
      }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the next window's frames have landed
    group_barrier();
  }
  if (ROLE == 0 && wave == 1 && g < NS) group_add_counters(c, counts, lane);
}

template <int KS>
__global__ __launch_bounds__(512) void wind_group_vocab_kernel(ModelDev m, CallDev c, GroupDev gd) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem_raw[];
  const int grp = (int)blockIdx.x % kGroups, g = (int)blockIdx.x / kGroups;   // workgroups go to the XCDs in turn
  if (grp >= gd.NG) return;
  if (blockIdx.x == 0 && threadIdx.x == 0) c.stats[kStatLoop] = (unsigned long long)wall_clock64();
  if (threadIdx.x < 256) vocab_loop<KS, 0>(m, c, gd, smem_raw, grp, g);
  else vocab_loop<KS, 1>(m, c, gd, smem_raw, grp, g);
}

}  // namespace wind
