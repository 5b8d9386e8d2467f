// The whole decode loop of a small batch as resident groups of workgroups, one group per XCD.
#pragma once
#include "wind_types.h"
#include "wind_decide_kernels.h"
#include "wind_group_protocol.h"
#include "wind_pred_kernels.h"

namespace wind {

// ---------------------------------------------------------------------------------------------
// Utterances are independent, so a batch needs no hand-over between the chip's eight XCDs: every XCD decodes
// its own utterances with a resident group of GW workgroups (one per CU), and what the group's
// workgroups tell each other stays in that XCD's L2.  A group holds up to four utterances at a time
// (slots); when one is done the slot takes the next of the group's list.  Utterances are dealt by falling
// length, back and forth over the slots.
//
// The weights the loop needs sit in registers, as matrix-core operands (all instances keep 70 to 131 scalars in lanes of vector
// registers): per workgroup CT parts of 32
// columns of W_out (waves 0-3, K split in four), the recurrent rows of UPW LSTM units and PPW rows of W_pred
// (waves 4-7, K split in four).  LDS holds the projected frames of the windows: two windows' worth per
// slot, loaded straight from memory a whole iteration before they are read.
//
// An iteration, and what bounds it (a chain of short steps; nothing here is long enough to be bound by bytes or flops):
//   waves 0-3  window rows as matrix-core operands from LDS, products with W_out, partial sums to LDS
//   all        keys of the workgroup's rows and columns -> exchange 1; every workgroup takes every slot's
//              decision from the keys (near-ties in fp32, only in rows before the first certain label)
//   waves 4-7  a label's LSTM step for this workgroup's units -> exchange 2 (hidden vector) -> projection
//              rows -> exchange 3 (projection); then, off the chain, the recurrent sums of the next step
//              and the frames of the window after next
// The three exchanges have no barrier and no flags: every 8-byte word carries its iteration (the keys: its
// parity), and a reader asks for the words it needs until all are this iteration's.  No word is overwritten before everybody
// has read it: new hidden vectors and projections come from every workgroup, so none can start a step that another has not
// finished.  Keys need not, and where some workgroup has none every workgroup also publishes the iterations it has decided
// (wind_group_protocol.h; looked at by a wave that idles during the window products.  Always doing so cost 2 to 6 %).
// Every wait is bounded: after spin_limit polls (the first one, for all to be on the chip: start_limit), or when the group's abort word is
// set, a wave sets that word and marks the workgroup failed, which then leaves at its next decision; the host
// then has the call decoded by the per-step kernels, or reports the error.
//
// How far an iteration looks (CallDev::W, the reach: frames of every slot) does not depend on the caller's window: a row tile has 16 rows,
// which its SPT slots share, and whether a frame's label is found by one iteration or by the next changes neither
// labels nor frames.  The counters stay those of windows of gd.win frames (group_outcome).  With several slots the group's workgroups
// are cut into RG = 2 row groups, each covering all columns with GW / 2 workgroups.  640 units, 1024 labels, lengths 200 .. 1500: 13 utterances
// (two slots), one tile of 2 x 8 rows 1.51 ms, two of 16 1.39; 20 (three slots), 3 x 5 rows 1.83, two tiles of 2 x 8 1.68, three
// of 16 1.73; 32 (four), 4 x 4 2.90, two tiles of 2 x 8 2.47, four of 16 2.63.  As many frames as the caller's
// window, before: one utterance of 1000 frames 2.94 / 1.26 / 0.98 / 0.84 ms at W = 1 / 4 / 8 / 16, now 0.84 at each (0.75 with kGroupOne).
// With three and four slots two tiles cost something where hardly any frame has a label and windows are long: 32 utterances at W = 16, four
// tiles of 16 rows / two of 2 x 8: 15 labels in 100 frames 2.61 / 2.45 ms, 6 1.82 / 1.75, 2 0.85 / 0.93, none 0.53 / 0.71.
template <int KS, int CT, int GW>
struct GroupCfg {
  static constexpr int H = 128 * KS;                      // = Hp = Hj
  static constexpr int UPW = H / GW, NR = 4 * UPW, PPW = H / GW;
  static constexpr int LT = NR / 16, PT = (PPW + 15) / 16;   // tiles of 16 weight rows
  static constexpr int QK = H / 4, QL = (QK + 63) / 64;      // a wave's quarter of K, and its loads per lane
  static constexpr int EST = H + 4, HST = H + 8;             // row strides in LDS (16 bytes of padding: banks)
  static constexpr int NI = (4 * CT + 7) / 8;                // (row quad, part) items of the key step per wave
  static_assert(H % GW == 0 && NR % 16 == 0, "units per workgroup");
  static constexpr size_t oE = 0;                                         // float [32][EST]
  static constexpr size_t oFred = oE + (size_t)32 * EST * 4;              // float [4][2 CT][4][80]
  static constexpr size_t oFbn = oFred + (size_t)4 * 2 * CT * 4 * 80 * 4; // float [4][2][16]
  static constexpr size_t oP = oFbn + 512;                                // float [slots][H]
  static constexpr size_t oHb = oP + (size_t)kGroupSlots * H * 4;         // bf16 [8][HST]
  static constexpr size_t oPred = oHb + (size_t)8 * HST * 2;              // float [4][16 PT][4]
  static constexpr size_t oRecp = oPred + (size_t)4 * 16 * PT * 4 * 4;    // float [4][NR][4]
  static constexpr size_t oRec = oRecp + (size_t)4 * NR * 4 * 4;          // float [slots][NR]
  static constexpr size_t oC = oRec + (size_t)kGroupSlots * NR * 4;       // float [slots][UPW]
  static constexpr size_t oW = oC + (size_t)kGroupSlots * UPW * 4;        // float [H] blank column of W_out
  static constexpr size_t oI = oW + (size_t)H * 4;                        // int stat[64], stat2[64], cnt[kNumStats], open windows [slots][2], fail, flags; float bp[UPW]
  static constexpr size_t oT = (oI + (64 + 64 + kNumStats + 2 * kGroupSlots + 2 + PPW) * 4 + 255) / 256 * 256;   // 256 bytes that group_touch writes to
  static constexpr size_t smem = oT + 256;
  static_assert(smem <= 160 * 1024, "LDS");
};

__device__ __forceinline__ unsigned long long group_ld(const unsigned long long *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// near: the readers share this CU's L2, a store need only reach that; else it goes to the memory side
__device__ __forceinline__ void group_st(unsigned long long *p, unsigned lo, unsigned hi, bool near) {
  const unsigned long long u = (unsigned long long)lo | ((unsigned long long)hi << 32);
  if (near) __hip_atomic_store(p, u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  else __hip_atomic_store(p, u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Workgroup barrier that waits for LDS only (outstanding loads and stores go on)
__device__ __forceinline__ void group_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}
// Whether every workgroup of the group has decided `need` iterations (progress: their counts, one word each, one line in all)
template <int GW>
__device__ __forceinline__ bool group_decided(const unsigned *progress, int lane, int need) {
  const unsigned v = lane < GW ? __hip_atomic_load(progress + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0x7FFFFFFFu;
  return (int)v >= need;
}
__device__ __forceinline__ void group_publish(unsigned *word, unsigned v, bool near) {
  if (near) __hip_atomic_store(word, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  else __hip_atomic_store(word, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// A quarter of a wait: asks again through `ask` (which returns whether this lane has all it needs) until every
// lane of the wave does.  False: gave up.
template <class Ask>
__device__ __forceinline__ bool group_poll(unsigned *abort_word, unsigned limit, const Ask &ask) {
  unsigned spins = 0;
  while (!__all(ask())) {
    if (++spins > limit || ((spins & 15u) == 0 && __hip_atomic_load(abort_word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))) {
      if ((threadIdx.x & 63) == 0) __hip_atomic_store(abort_word, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      return false;
    }
  }
  return true;
}
// 64 lanes x 16 bytes from memory to 1 KB of LDS.  Written as assembly so that the compiler does not make later LDS
// reads of this wave wait for it: whoever reads the rows is a barrier and an explicit wait away.
__device__ __forceinline__ void group_load_lds(const void *src, unsigned lds) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(lds), "v"(src) : "memory");
}

// Load time: the state after the start token (its LSTM step from zero, projection, recurrent sums of the next
// step), the same for every utterance.  Workgroup = 4 rows of [w_hh ; w_pred], one per wave.
template <class WT>
__global__ __launch_bounds__(256) void group_start_kernel(ModelDev m, float *start_c, float *start_p, float *start_rec) {
  extern __shared__ float hs[];
  const int Hp = m.Hp, tid = threadIdx.x;
  for (int u = tid; u < Hp; u += 256) {
    const float4 x = *reinterpret_cast<const float4 *>(m.emb_gates + (size_t)m.V * 4 * Hp + 4 * u);
    const float ig = 1.f / (1.f + expf(-x.x)), og = 1.f / (1.f + expf(-x.w));
    const float cn = ig * tanhf(x.z);
    hs[u] = og * tanhf(cn);
    if (blockIdx.x == 0) start_c[u] = cn;
  }
  __syncthreads();
  const int lane = tid & 63, row = (int)blockIdx.x * 4 + (tid >> 6);
  if (row >= 4 * Hp + m.Hj) return;
  const WT *w = row < 4 * Hp ? reinterpret_cast<const WT *>(m.w_cat[0]) + (size_t)row * Hp
                             : reinterpret_cast<const WT *>(m.w_pred) + (size_t)(row - 4 * Hp) * Hp;
  float a = 0.f;
  for (int k = 2 * lane; k < Hp; k += 128) {
    const float2 x = ldw2(w, k);
    a = fmaf(x.x, hs[k], a);
    a = fmaf(x.y, hs[k + 1], a);
  }
  a = wave_sum(a);
  if (lane == 0) {
    if (row < 4 * Hp) start_rec[row] = a;
    else start_p[row - 4 * Hp] = a + m.b_pred[row - 4 * Hp];
  }
}

// What the host reads after the loop, in one launch, straight into pinned memory; the call's number last: the host
// watches for it instead of waiting for the stream (a wait costs 10 us and more after the work is done, and events between the
// kernels 6 us each; the call's times are the device's time stamps).
__global__ __launch_bounds__(128) void group_collect_kernel(const int *n_active, const unsigned *bar, int NX, const unsigned long long *stats,
                                                            int *h_flag, unsigned long long *h_stats, int number) {
  const int i = threadIdx.x;
  if (i == 0) {
    unsigned gave_up = 0u, near = 2u;
    for (int g = 0; g < NX; ++g) {
      gave_up |= bar[g * kGroupBarInts];
      near = min(near, bar[g * kGroupBarInts + 1]);
    }
    h_flag[0] = n_active[0];
    h_flag[1] = (int)gave_up;
    h_flag[2] = (int)near;
  }
  if (i < kStatWords) h_stats[i] = i == kStatEnd ? (unsigned long long)wall_clock64() : stats[i];
  __threadfence_system();
  __syncthreads();
  if (i == 0) __hip_atomic_store(h_flag + 8, number, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// 64 lanes x 4 bytes to LDS nobody reads: brings the lines they lie in into this CU's cache
__device__ __forceinline__ void group_touch(const void *src, unsigned lds) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, off" ::"s"(lds), "v"(src) : "memory");
}

// The part of the loop's state that every wave keeps for itself: lane a holds slot a.
struct GroupLane {
  int b, t, len, sym, cnt;   // utterance, frame, length, labels on the frame, labels so far (len = t = 0: slot empty)
  int rpos;                  // t modulo 2 W: the frame's row in its ring of projected frames
  int ld0, ld;               // frames loaded (or asked for) before the last decision, and now
  int nb, nlen, round;       // the slot's next utterance (-1: none)
};
// Calls with a group per utterance (up to 8 utterances) take instances of their own, without all that is there for several slots and for a
// slot's next utterance: 640 units keep 105 scalars in lanes of vector registers instead of 136, and one utterance of 1000 frames
// takes 749 instead of 837 us; fp32 models of 128 units and 128 labels keep no vector register in scratch memory (53, the weights
// of W_out among them) and 500 frames take 807 instead of 1084 us.  Asynchronous calls that may stop short, whose windows of the caller's size
// are counted to max_iters in every wave, have such instances too.
enum { kGroupMany, kGroupOne, kGroupLimited };

// What the caller's windows have come to in a slot.  In limited calls (LIM) every wave keeps it, since all have to stop at the same frame; else
// it is in LDS, where only the wave that counts looks at it.
struct GroupOpen {
  int wc;   // windows of the caller's size so far
  int ph;   // blank frames of the open one that earlier iterations have seen (0: none is open)
};

// The entry of order `round` of this lane's slot: utterances by falling length, dealt back and forth over the slots.
__device__ __forceinline__ void group_next(const CallDev &c, const GroupDev &gd, int grp, int lane, int n_order, int round, int &b, int &len) {
  const int VS = gd.NG * gd.NS, v = lane * gd.NG + grp, rank = round * VS + ((round & 1) ? VS - 1 - v : v);
  b = -1;
  len = 0;
  if (lane < gd.NS && rank < n_order) {
    b = gd.order[rank];
    len = c.len[b];
  }
}
// ONE: a group per utterance, no slot has a next one
template <bool ONE>
__device__ __forceinline__ GroupLane group_first_slots(const CallDev &c, const GroupDev &gd, int grp, int lane, int n_order) {
  GroupLane sl;
  group_next(c, gd, grp, lane, n_order, 0, sl.b, sl.len);
  if constexpr (ONE) sl.nb = -1, sl.nlen = 0;
  else group_next(c, gd, grp, lane, n_order, 1, sl.nb, sl.nlen);
  sl.t = sl.sym = sl.cnt = sl.rpos = sl.ld0 = 0;
  sl.round = 1;
  if (sl.b < 0) sl.b = 0;
  sl.ld = min(sl.len, 2 * c.W);
  return sl;
}

// Frames of the slot's window in this iteration: up to c.W, the reach (see group_shape), which may hold several windows of the caller's
// size, gd.win, or end inside one; no more of those than the call may take.
template <bool LIM>
__device__ __forceinline__ int group_window(const CallDev &c, const GroupDev &gd, const GroupLane &sl, const GroupOpen &open) {
  const int n = min(c.W, sl.len - sl.t);
  return LIM ? min(n, gd.win * min(gd.max_iters - open.wc, kGroupMaxW) - open.ph) : n;
}

// The frames that the slots of row tile rt have come to need (from ld0 to ld), into their rings of 2 W rows, one frame per wave
// in turn (part of nparts).
template <int H, int EST>
__device__ __forceinline__ void group_load_frames(const CallDev &c, const GroupDev &gd, const GroupLane &sl, const float *ecache, int rt, int lane,
                                                  int part, int nparts) {
  const unsigned lds0 = (unsigned)(unsigned long long)(__attribute__((address_space(3))) const float *)ecache;
  const int W2 = 2 * c.W;
  for (int q = 0; q < gd.SPT; ++q) {
    const int a = rt * gd.SPT + q;
    if (a >= gd.NS) break;
    const int f0 = __builtin_amdgcn_readlane(sl.ld0, a), f1 = __builtin_amdgcn_readlane(sl.ld, a);
    const int t = __builtin_amdgcn_readlane(sl.t, a), rp = __builtin_amdgcn_readlane(sl.rpos, a), b = __builtin_amdgcn_readlane(sl.b, a);
    for (int f = f0 + ((part - f0) & (nparts - 1)); f < f1; f += nparts) {
      int rr = rp + (f - t);
      if (rr >= W2) rr -= W2;
      const float *src = c.e + (size_t)((unsigned)b * (unsigned)c.T + (unsigned)f) * H + lane * 4;
      const unsigned dst = lds0 + (unsigned)(q * W2 + rr) * (EST * 4);
#pragma unroll
      for (int i = 0; i < (H + 255) / 256; ++i)
        if (i * 256 + lane * 4 < H) group_load_lds(src + i * 256, dst + i * 1024);
    }
  }
}

// What a decided iteration does to the slots, in every wave alike: m_nb = rows of the group whose label is not blank, lab = row
// `lane`'s label, need = rows that were decided again in fp32.  `writer` (one wave of the group) writes the outputs and
// counts.  Returns whether this lane's slot takes an LSTM step (for tok) and whether it took a new utterance.
template <bool LIM, bool ONE>
__device__ __forceinline__ void group_outcome(const CallDev &c, const GroupDev &gd, GroupLane &sl, GroupOpen &open, int grp, int lane, int n_order, int nwin, int V,
                                              unsigned long long m_nb, unsigned long long need, int lab, bool writer, int *counts, int &tok,
                                              bool &emits, bool &fresh_slot) {
  const int W = c.W, W2 = 2 * W, oshift = lane < gd.NS ? lane * W : 0;
  const unsigned segm = (1u << W) - 1u;
  const unsigned seg = lane < gd.NS ? (unsigned)(m_nb >> oshift) & segm : 0u;
  const int first = seg ? __ffs((int)seg) - 1 : -1;
  if constexpr (ONE) tok = __builtin_amdgcn_readlane(lab, max(__builtin_amdgcn_readfirstlane(first), 0));   // only lane 0 has a slot
  else tok = __shfl(lab, oshift + max(first, 0), kWave);
  tok = min(max(tok, 0), V);
  emits = false;
  fresh_slot = false;
  if (nwin > 0) {
    const int t0 = sl.t;
    const WindowOutcome wo = window_outcome(c, make_int4(sl.b, sl.t, sl.len, sl.sym), sl.cnt, nwin, first, tok, V, 0, writer);
    const int adv = wo.slot.y - sl.t;
    sl.t = wo.slot.y; sl.sym = wo.slot.w; sl.cnt = wo.cnt;
    sl.rpos += adv;
    if (sl.rpos >= W2) sl.rpos -= W2;
    sl.ld0 = sl.ld;
    sl.ld = max(sl.ld, min(sl.len, sl.t + W2));
    bool cut = false;
    if (writer || LIM) {   // behind the state that everybody waits for: 50 ns of an iteration where every wave did this first
      // What that is in windows of the caller's size, which start where the last label or the last whole window left off: `full` blank ones,
      // and one that a label or the last frame closes, `rem` blank frames into it, or that stays open
      unsigned at0 = (unsigned)(unsigned long long)(__attribute__((address_space(3))) int *)counts;
      asm volatile("" : "+v"(at0));   // formed here: the compiler keeps addresses that do not change in registers over the loop
      const auto kept = (__attribute__((address_space(3))) int *)(at0 + (kNumStats + 2 * lane) * 4);
      if constexpr (!LIM) open = GroupOpen{kept[0], kept[1]};
      const int seen = open.ph + (first < 0 ? nwin : first), full = (int)(((unsigned)seen * gd.win_inv) >> 16), rem = seen - full * gd.win;
      const bool closes = first >= 0 || (rem > 0 && t0 + nwin == sl.len);
      const int n_last = first < 0 ? rem : min(gd.win, sl.len - (t0 + first - rem));
      const int looked = first < 0 ? W : min(W, (full + 1) * gd.win - open.ph);   // rows of the frames up to the end of the window that decided
      const int rech = __popc((unsigned)(need >> oshift) & segm & ((1u << looked) - 1u));
      open.wc += full + closes;
      open.ph = closes ? 0 : rem;
      if constexpr (LIM) cut = (wo.flag & 1) && open.wc >= gd.max_iters;
      else {   // the slot's next utterance starts from zero
        kept[0] = wo.flag & 1 ? open.wc : 0;
        kept[1] = wo.flag & 1 ? open.ph : 0;
      }
      if (writer) {
        // The call's counters (32 bits each).  LDS additions that nobody waits for, written as assembly: the
        // compiler turns an atomicAdd of several lanes into a loop over them, half a microsecond for all of these.
        const unsigned ev = wo.ev, forced = (ev >> 29) & 1u;
        auto add = [&](int which, unsigned v) { asm volatile("ds_add_u32 %0, %1" ::"v"(at0 + 4 * which), "v"(v) : "memory"); };
        const int blanks = full * gd.win;
        add(ST_WINDOWS, (unsigned)(full + closes));
        add(ST_ROWS, (unsigned)(blanks + (closes ? n_last : 0)));
        add(ST_USEFUL, (unsigned)(blanks + (first >= 0 ? rem + 1 : closes ? rem : 0)));
        add(ST_RECHECK, (unsigned)rech);
        add(ST_LABELS, (ev >> 28) & 1u);
        add(ST_FORCED, forced);
        add(ST_OVERFLOW, (ev >> 30) & 1u);
        add(kStatJump0 + gd.win, (unsigned)full);
        add(kStatJump0 + rem + (int)forced, closes ? 1u : 0u);
        // no branch on the condition that decides below: the compiler would make two of that branch, with all of the state copied in each
        asm volatile("ds_max_u32 %0, %1" ::"v"(at0 + 4 * ST_ITER), "v"((wo.flag & 1) && !cut ? 0 : open.wc) : "memory");
        if (LIM && cut) atomicAdd(&c.n_active[0], 1);
      }
    }
    const bool done = !(wo.flag & 1) || cut;
    emits = (wo.flag & 2) && !done;
    if (done) {   // the slot's next utterance, or nothing
      fresh_slot = !ONE && sl.nb >= 0;
      sl.b = fresh_slot ? sl.nb : 0;
      sl.len = fresh_slot ? sl.nlen : 0;
      sl.t = sl.sym = sl.cnt = sl.rpos = sl.ld0 = 0;
      if constexpr (LIM) open = GroupOpen{0, 0};
      sl.ld = min(sl.len, W2);
      if (fresh_slot) {
        ++sl.round;
        group_next(c, gd, grp, lane, n_order, sl.round, sl.nb, sl.nlen);
      }
    }
  } else {
    sl.ld0 = sl.ld;
  }
}
__device__ __forceinline__ void group_add_counters(const CallDev &c, const int *counts, int lane) {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // this wave's additions are in
  for (int j = lane; j < kNumStats; j += 64) {
    if (j == ST_ITER) atomicMax(&c.stats[j], (unsigned long long)counts[j]);
    else if (counts[j]) atomicAdd(&c.stats[j], (unsigned long long)counts[j]);
  }
}

template <int KS, int CT, int GW, int MODE, int ROLE>
__device__ __forceinline__ void group_loop(const ModelDev &m, const CallDev &c, const GroupDev &gd, unsigned char *smem, int grp, int g) {
  using Cfg = GroupCfg<KS, CT, GW>;
  constexpr int H = Cfg::H, NR = Cfg::NR, QK = Cfg::QK, QL = Cfg::QL;
  constexpr bool ONE = MODE != kGroupMany, LIM = MODE == kGroupLimited;
  constexpr int SL = ONE ? 1 : kGroupSlots;
  float *ecache = reinterpret_cast<float *>(smem + Cfg::oE), *fred = reinterpret_cast<float *>(smem + Cfg::oFred);
  float *fbn = reinterpret_cast<float *>(smem + Cfg::oFbn), *pfull = reinterpret_cast<float *>(smem + Cfg::oP);
  bf16_t *hbuf = reinterpret_cast<bf16_t *>(smem + Cfg::oHb);
  float *predp = reinterpret_cast<float *>(smem + Cfg::oPred), *recp = reinterpret_cast<float *>(smem + Cfg::oRecp);
  float *recs = reinterpret_cast<float *>(smem + Cfg::oRec), *cst = reinterpret_cast<float *>(smem + Cfg::oC);
  float *wbl = reinterpret_cast<float *>(smem + Cfg::oW);
  int *stat = reinterpret_cast<int *>(smem + Cfg::oI), *stat2 = stat + 64, *counts = stat2 + 64, *fail = counts + kNumStats + 2 * kGroupSlots, *near_w = fail + 1;
  float *bpl = reinterpret_cast<float *>(near_w + 1);   // this workgroup's rows of b_pred

  int lane = threadIdx.x & 63, tid1 = threadIdx.x & 255, l15 = lane & 15, l4 = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), w4 = wave & 3;   // w4: the wave's quarter of K
  const int W = c.W, V = m.V, NS = gd.NS, SPT = gd.SPT, W2 = 2 * W, R = NS * W, nparts = c.nparts_tiny, kstride = nparts + 1;
  const int CG = GW / gd.RG, rt = g / CG, cg = g - rt * CG;
  unsigned *abort_word = gd.bar + grp * kGroupBarInts;
  unsigned long long *hx = gd.h_x + (size_t)grp * kGroupSlots * H, *px = gd.p_x + (size_t)grp * kGroupSlots * H;
  unsigned long long *kbase = gd.keys + (size_t)grp * 2 * kGroupRows * kstride;
  const int unit0 = g * Cfg::UPW, prow0 = g * Cfg::PPW;

  // ---- the slots' first utterances
  const int n_order = *gd.n_order;
  GroupLane sl = group_first_slots<ONE>(c, gd, grp, lane, n_order);
  GroupOpen open{0, 0};

  // ---- weights into registers
  bf16x8 wo[ROLE == 0 ? 2 * CT : 1][KS];                                   // W_out columns
  bf16x8 wr[ROLE == 1 ? Cfg::LT : 1][KS], wp[ROLE == 1 ? Cfg::PT : 1][KS];   // recurrent rows, projection rows
  if constexpr (ROLE == 0) {
#pragma unroll
    for (int t = 0; t < 2 * CT; ++t) {
      const int col = min(((t >> 1) * CG + cg) * 32 + 16 * (t & 1) + l15, m.Vpad - 1);
      const bf16_t *src = reinterpret_cast<const bf16_t *>(m.w_out) + (size_t)col * H + w4 * QK + l4 * 8;
#pragma unroll
      for (int i = 0; i < KS; ++i) wo[t][i] = *reinterpret_cast<const bf16x8 *>(src + i * 32);
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
      const bf16_t *src = reinterpret_cast<const bf16_t *>(m.w_pred) + (size_t)(prow0 + min(16 * t + l15, Cfg::PPW - 1)) * H + w4 * QK + l4 * 8;
#pragma unroll
      for (int i = 0; i < KS; ++i) wp[t][i] = *reinterpret_cast<const bf16x8 *>(src + i * 32);
    }
  }

  auto load_frames = [&]() { group_load_frames<H, Cfg::EST>(c, gd, sl, ecache, rt, lane, w4, 4); };

  // ---- state after the start token
  if constexpr (ROLE == 0) {
    for (int i = tid1; i < NS * H; i += 256) pfull[i] = m.start_p[i % H];
    for (int i = tid1; i < H; i += 256) wbl[i] = m.w_blank[i];
    if (tid1 == 0) *fail = 0;
  } else {
    for (int i = tid1; i < NS * NR; i += 256) recs[i] = m.start_rec[unit0 * 4 + i % NR];
    for (int i = tid1; i < NS * Cfg::UPW; i += 256) cst[i] = m.start_c[unit0 + i % Cfg::UPW];
    for (int i = tid1; i < kNumStats + 2 * kGroupSlots; i += 256) counts[i] = 0;
    if (tid1 < Cfg::PPW) bpl[tid1] = m.b_pred[prow0 + tid1];
    load_frames();
  }
  // ---- where the workgroups sit: XCD numbers, exchanged with device-wide stores
  if (wave == 0) {
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
      *near_w = (same ? 1 : 0) | (group_keys_suffice(nparts, CG, gd.RG) ? 0 : 2);
      if (!got) *fail = 1;
      if (g == 0) abort_word[1] = same ? 2u : 1u;
    }
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  group_barrier();
  const int flags = __builtin_amdgcn_readfirstlane(*near_w);   // one register for both
  const bool near = flags & 1, publishes = flags & 2;

  // ---- constants of this lane's places in the steps below
  const float b_blank = m.b_out[V];
  // the blank column's part that this lane needs (the row's LDS reads bound that step)
  float4 breg[ROLE == 0 ? KS : 1][2];
  if constexpr (ROLE == 0) {
#pragma unroll
    for (int i = 0; i < KS; ++i)
#pragma unroll
      for (int h = 0; h < 2; ++h) breg[i][h] = *reinterpret_cast<const float4 *>(wbl + w4 * QK + l4 * 8 + i * 32 + 4 * h);
  }
  const unsigned touch_lds = (unsigned)(unsigned long long)(__attribute__((address_space(3))) unsigned char *)(smem + Cfg::oT);
  const unsigned winv = 65536u / (unsigned)W + 1u;   // x / W for x < 64
  auto div_w = [&](int x) { return (int)(((unsigned)x * winv) >> 16); };
  float bias[Cfg::NI][2];
#pragma unroll
  for (int k = 0; k < Cfg::NI; ++k)
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const int item = wave + 8 * k, part = (item >> 2) * CG + cg, col = part * 32 + 16 * t + l15;
      bias[k][t] = item < 4 * CT && part < nparts && col < V ? m.b_out[col] : kKeyNone;   // what is added to kKeyNone vanishes in it
    }
  int pend = 0, pend_slot[kGroupSlots] = {0, 0, 0, 0};   // ROLE 1: slots whose recurrent sums wait for their partial sums

  for (int it = 0;; ++it) {
    // opaque: what follows from the lane's number is formed again in every iteration, where it is used, instead of being kept
    // in registers over the loop (the weights need them)
    asm volatile("" : "+v"(lane), "+v"(tid1));
    l15 = lane & 15;
    l4 = lane >> 4;
    const int nwin = group_window<LIM>(c, gd, sl, open);   // lanes of empty slots: 0
    if (!__any(nwin > 0)) break;
    const int tag = group_key_tag(it);
    const unsigned stamp = (unsigned)it + 1u;
    unsigned long long *kp = kbase + (size_t)group_key_buffer(it) * kGroupRows * kstride;
    if constexpr (ROLE == 1) {
      // the keys that this iteration's replace have been read by everybody: nearly always so at once, and looked at while waves 0-3
      // form the window products
      if (publishes && wave == 6 && group_keys_need(it) > 0 &&
          !group_poll(abort_word, gd.spin_limit, [&]() { return group_decided<GW>(abort_word + 32, lane, group_keys_need(it)); }) && lane == 0) *fail = 1;
    }
    if constexpr (ROLE == 0) {
      // ---- window rows as matrix-core operands: lane (row l15, K group l4) takes 8 consecutive frames' projections
      // per step of 32 of this wave's quarter of K, adds the prediction projection, applies the ReLU and rounds:
      // its part of the first operand of a 16 x 16 x 32 product.  Blank logit and squared norm in fp32.
      f32x4 acc[2 * CT];
#pragma unroll
      for (int t = 0; t < 2 * CT; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
      const int gq = div_w(l15), gl = gq < SPT ? gq : 0, gj = gq < SPT ? l15 - gl * W : 0;   // row l15 of the tile: slot, row of its window
      const int ga = min(rt * SPT + gl, NS - 1), gloc = max(ga - rt * SPT, 0);
      int rr = (ONE ? __builtin_amdgcn_readfirstlane(sl.rpos) : __shfl(sl.rpos, ga, kWave)) + gj;
      if (rr >= W2) rr -= W2;
      const float *er = ecache + (gloc * W2 + rr) * Cfg::EST + w4 * QK + l4 * 8;
      const float *pr = pfull + ga * H + w4 * QK + l4 * 8;
      float dot = 0.f, nrm = 0.f;
      // the LDS operands of a step are read one step ahead, into registers that take turns
      float4 eo[2][2], po[2][2];
      auto read_ops = [&](int set, int i) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          eo[set][h] = *reinterpret_cast<const float4 *>(er + i * 32 + 4 * h);
          po[set][h] = *reinterpret_cast<const float4 *>(pr + i * 32 + 4 * h);
        }
      };
      read_ops(0, 0);
#pragma unroll
      for (int i = 0; i < KS; ++i) {
        if (i + 1 < KS) read_ops((i + 1) & 1, i + 1);
        float x[8], d = 0.f;   // the blank logit's sum in blocks of 8 products, a step's: as short as the other kernels' (lanes and a tree)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const float4 e4 = eo[i & 1][h], p4 = po[i & 1][h], b4 = breg[i][h];
          float *y = x + 4 * h;
          y[0] = fmaxf(e4.x + p4.x, 0.f); y[1] = fmaxf(e4.y + p4.y, 0.f); y[2] = fmaxf(e4.z + p4.z, 0.f); y[3] = fmaxf(e4.w + p4.w, 0.f);
          d = fmaf(y[0], b4.x, d); d = fmaf(y[1], b4.y, d); d = fmaf(y[2], b4.z, d); d = fmaf(y[3], b4.w, d);
          nrm = fmaf(y[0], y[0], nrm); nrm = fmaf(y[1], y[1], nrm); nrm = fmaf(y[2], y[2], nrm); nrm = fmaf(y[3], y[3], nrm);
        }
        dot += d;
        const u32x4 zu = u32x4{pack_bf16x2(x[0], x[1]), pack_bf16x2(x[2], x[3]), pack_bf16x2(x[4], x[5]), pack_bf16x2(x[6], x[7])};
#pragma unroll
        for (int t = 0; t < 2 * CT; ++t) acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, zu), wo[t][i], acc[t], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);   // keeps the reads at one step ahead: registers
      }
      dot = quarter_sum(dot);
      nrm = quarter_sum(nrm);
      // register r of lane l: row 4 l4 + r, column l15 of tile t; 80 floats per r: the readers below hit different banks
#pragma unroll
      for (int t = 0; t < 2 * CT; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) fred[((w4 * 2 * CT + t) * 4 + r) * 80 + lane] = acc[t][r];
      if (lane < 16) {
        fbn[(w4 * 2 + 0) * 16 + lane] = dot;
        fbn[(w4 * 2 + 1) * 16 + lane] = nrm;
      }
    }
    group_barrier();   // B1: partial sums of the logits (and, from the last step, of the recurrent rows) are in LDS
    // ---- keys: item (row quad q4, part): lane = (row 4 q4 + l4, columns l15 and l15 + 16 of the part)
#pragma unroll
    for (int k = 0; k < Cfg::NI; ++k) {
      const int item = wave + 8 * k;
      if (item >= 4 * CT) continue;
      const int q4 = item & 3, ct = item >> 2, part = ct * CG + cg;
      float k1 = kKeyNone, k2 = kKeyNone;
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        float v = bias[k][t];
#pragma unroll
        for (int w = 0; w < 4; ++w) v += fred[((w * 2 * CT + 2 * ct + t) * 4 + l4) * 80 + 16 * q4 + l15];
        push_top2(k1, k2, make_key(v, 16 * t + l15));
      }
      merge_top2(k1, k2, dpp_f32<kDppRowMirror>(k1), dpp_f32<kDppRowMirror>(k2));
      merge_top2(k1, k2, dpp_f32<kDppRowHalfMirror>(k1), dpp_f32<kDppRowHalfMirror>(k2));
      merge_top2(k1, k2, dpp_f32<kDppQuadXor2>(k1), dpp_f32<kDppQuadXor2>(k2));
      merge_top2(k1, k2, dpp_f32<kDppQuadXor1>(k1), dpp_f32<kDppQuadXor1>(k2));
      const int lr = 4 * q4 + l4, row = rt * SPT * W + lr;
      if (part < nparts && l15 == 0 && lr < SPT * W && row < R)
        group_st(kp + (size_t)row * kstride + part, __float_as_uint(k1), __float_as_uint(key_with_tag(k2, tag)), near);
    }
    if constexpr (ROLE == 1) {
      if (wave == 4 && cg == 0 && lane < SPT * W && rt * SPT * W + lane < R) {   // SPT * W <= 16
        auto sum4 = [&](int which) {
          return (fbn[(0 + which) * 16 + lane] + fbn[(2 + which) * 16 + lane]) + (fbn[(4 + which) * 16 + lane] + fbn[(6 + which) * 16 + lane]);
        };
        const float d2 = sum4(0) + b_blank, n2 = sum4(1);
        group_st(kp + (size_t)(rt * SPT * W + lane) * kstride + nparts, __float_as_uint(d2), __float_as_uint(key_with_tag(sqrtf(n2), tag)), near);
      }
      for (int i = tid1; i < pend * NR; i += 256) {
        const int e = i / NR, row = i - e * NR;
        float v = 0.f;
#pragma unroll
        for (int w = 0; w < 4; ++w) v += recp[(w * NR + row) * 4 + e];
        const int s = e == 0 ? pend_slot[0] : e == 1 ? pend_slot[1] : e == 2 ? pend_slot[2] : pend_slot[3];
        recs[s * NR + row] = v;
      }
      pend = 0;
    }
    if constexpr (ROLE == 1) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the last iteration's frames have landed
    // ---- exchange 1: four rows per wave, 16 lanes per row, lane s with the keys of parts s and s + 16
    if (4 * wave < R) {
      const int row = 4 * wave + l4, a = div_w(row);
      const bool valid = ONE ? row < __builtin_amdgcn_readfirstlane(nwin) : row - a * W < __shfl(nwin, a, kWave);   // one slot: no row past its window
      float2 kA = make_float2(kKeyNone, kKeyNone), kB = kA, kC = make_float2(0.f, 0.f);
      auto pair = [](unsigned long long u) { return make_float2(__uint_as_float((unsigned)u), __uint_as_float((unsigned)(u >> 32))); };
      const unsigned long long *kr = kp + (size_t)row * kstride;
      const bool got = group_poll(abort_word, gd.spin_limit, [&]() {
        if (!valid) return true;
        if (l15 < nparts) kA = pair(group_ld(kr + l15));
        if (l15 + 16 < nparts) kB = pair(group_ld(kr + l15 + 16));
        kC = pair(group_ld(kr + nparts));
        return (l15 >= nparts || key_tag(kA.y) == tag) && (l15 + 16 >= nparts || key_tag(kB.y) == tag) && key_tag(kC.y) == tag;
      });
      if (!got && lane == 0) *fail = 1;
      const float a2 = l15 < nparts ? key_with_tag(kA.y, 0) : kKeyNone, b2 = l15 + 16 < nparts ? key_with_tag(kB.y, 0) : kKeyNone;
      const float kbest = row16_max_f32(fmaxf(kA.x, kB.x));
      const float vbest = key_val(kbest), top = fmaxf(vbest, kC.x);
      const float thresh = top - (m.tau_scale * kC.y + 6.2e-5f * fabsf(top));
      const int cnt = row16_sum_i32((key_val(kA.x) >= thresh) + (key_val(a2) >= thresh) + (key_val(kB.x) >= thresh) + (key_val(b2) >= thresh));
      int col = -1;
      if (kA.x == kbest) col = l15 * 32 + key_col(kbest);
      if (kB.x == kbest) col = (l15 + 16) * 32 + key_col(kbest);
      col = row16_max_i32(col);
      int label = V;
      if (valid && !(vbest < thresh)) label = cnt == 1 && kC.x < thresh ? col : -1;   // -1: near-tie
      if (l15 == 0) stat[row] = label;
      // The step of a label starts with its row of input sums, from a table that no L2 holds: a row that may be the window's first
      // label asks for its lines now, while the decision is completed (step 0.94 -> 0.7 us).  The
      // column is clamped: with NaN logits no key is a label's
      if (label != V && l15 < (NR * 4 + 127) / 128 + 1)
        group_touch(m.emb_gates + (unsigned)min(max(col, 0), V) * (4u * H) + (unsigned)(unit0 * 4 + min(l15 * 32, NR - 1)), touch_lds);
    }
    group_barrier();   // B2: every row's label, or that it is a near-tie
    if (*fail) return;
    int lab = lane < R ? stat[lane] : V;
    unsigned long long m_nb = __ballot(lab >= 0 && lab != V);
    // near-ties before the first certain label of their window: fp32 logits, one row per wave
    const int oa = div_w(lane), oj = lane - oa * W;
    const unsigned long long need = __ballot(lab < 0 && ((m_nb >> (oa * W)) & ((1ull << oj) - 1ull)) == 0ull);
    if (need) {
      unsigned long long todo = need;
      // the waves with the fuller registers leave these to the others
      constexpr bool mine = ROLE == 0 || NR <= 80;
      constexpr int turns = NR <= 80 ? 8 : 4;
      for (int k = 0; mine && todo; ++k, todo &= todo - 1) {
        if ((k & (turns - 1)) != (wave & (turns - 1))) continue;
        const int row = __builtin_amdgcn_readfirstlane(__ffsll((long long)todo) - 1), a = __builtin_amdgcn_readlane(oa, row), j = __builtin_amdgcn_readlane(oj, row);
        const int b = __builtin_amdgcn_readlane(sl.b, a), t = __builtin_amdgcn_readlane(sl.t, a);
        float4 kk0 = no_keys();
        const unsigned long long *kr = kp + (size_t)row * kstride;
        const unsigned long long uc = group_ld(kr + nparts);
        if (lane < nparts) {
          const unsigned long long u = group_ld(kr + lane);
          kk0.x = __uint_as_float((unsigned)u);
          kk0.y = key_with_tag(__uint_as_float((unsigned)(u >> 32)), 0);
        }
        const float vblank = __uint_as_float((unsigned)uc), znorm = __uint_as_float((unsigned)(uc >> 32));
        const float top = fmaxf(key_val(wave_max_f32(kk0.x)), vblank);
        const float thresh = top - (m.tau_scale * znorm + 6.2e-5f * fabsf(top));
        CallDev cl = c;
        cl.p = pfull + ((long long)a - b) * H;   // recheck_row looks at row b
        int none = -1;
        float unused = 0.f;
        const int l = recheck_row<KS, 2>(m, cl, row, b, t + j, nparts, nparts, 32, vblank, thresh, kk0, false, no_keys(), false, none, unused);
        if (lane == 0) stat2[row] = l;
      }
      group_barrier();
      if ((need >> lane) & 1ull) lab = stat2[lane];
      m_nb = __ballot(lab >= 0 && lab != V);
    }
    if (ROLE == 1 && publishes && wave == 6 && lane == 0) group_publish(abort_word + 32 + g, stamp, near);   // this workgroup's reads of the keys are done
    // ---- outcome of every slot's window; one wave of workgroup 0 writes the outputs
    int tok;
    bool emits, fresh_slot;
    group_outcome<LIM, ONE>(c, gd, sl, open, grp, lane, n_order, nwin, V, m_nb, need, lab, ROLE == 1 && wave == 7 && g == 0, counts, tok, emits, fresh_slot);
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
      // ---- LSTM step: thread (emitting slot le, gate row li of this workgroup's units); waves 0-3 first, which get here earlier
      const int lvt = ROLE == 0 ? tid1 : tid1 + 256, le = lvt / NR, li = lvt - le * NR;
      if (le < n_em) {
        const int s = le == 0 ? es[0] : le == 1 ? es[1] : le == 2 ? es[2] : es[3], tk = le == 0 ? et[0] : le == 1 ? et[1] : le == 2 ? et[2] : et[3];
        const float pre = recs[s * NR + li] + m.emb_gates[(unsigned)tk * (4u * H) + (unsigned)(unit0 * 4 + li)];   // fits 32 bits: checked by the host
        const float act = (li & 3) == 2 ? tanhf(pre) : 1.f / (1.f + expf(-pre));
        const float ig = dpp_f32<0x00>(act), fg = dpp_f32<0x55>(act), gg = dpp_f32<0xAA>(act), og = dpp_f32<0xFF>(act);   // the unit's four gates
        if ((li & 3) == 0) {
          const int u = li >> 2;
          const float cn = fg * cst[s * Cfg::UPW + u] + ig * gg;
          cst[s * Cfg::UPW + u] = cn;
          const float hv = og * tanhf(cn);
          const unsigned hb = f32_to_bf16_bits(hv), lb = f32_to_bf16_bits(hv - bf16_bits_to_f32(hb));
          group_st(hx + s * H + unit0 + u, hb | (lb << 16), stamp, near);
        }
      }
      if constexpr (ROLE == 1) {
        // ---- exchange 2: this wave's quarter of the new hidden vectors, as bf16 hi and lo rows
        unsigned long long u[SL][QL];
        const bool got = group_poll(abort_word, gd.spin_limit, [&]() {
#pragma unroll
          for (int e = 0; e < SL; ++e)
            if (e < n_em) {
#pragma unroll
              for (int q = 0; q < QL; ++q) u[e][q] = group_ld(hx + es[e] * H + w4 * QK + min(lane + 64 * q, QK - 1));
            }
          bool fresh = true;
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
              if (lane + 64 * q < QK) {
                bf16_t *d = hbuf + 2 * e * Cfg::HST + w4 * QK + lane + 64 * q;
                d[0] = (bf16_t)u[e][q];
                d[Cfg::HST] = (bf16_t)(u[e][q] >> 16);
              }
          }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // this wave's own rows: no barrier
        bf16x8 hf[KS];   // first operand: rows 2 e and 2 e + 1 = hi and lo of the e-th emitting slot (rows of others: not looked at)
        const bf16_t *hsrc = hbuf + (l15 & 7) * Cfg::HST + w4 * QK + l4 * 8;
#pragma unroll
        for (int i = 0; i < KS; ++i) hf[i] = *reinterpret_cast<const bf16x8 *>(hsrc + i * 32);
        f32x4 pacc[Cfg::PT];
#pragma unroll
        for (int t = 0; t < Cfg::PT; ++t) {
          pacc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int i = 0; i < KS; ++i) pacc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(hf[i], wp[t][i], pacc[t], 0, 0, 0);
          // lane (weight row l15, first-operand rows 4 l4 ..): slots 2 l4 and 2 l4 + 1, hi + lo
          if (lane < 32)
            *reinterpret_cast<float2 *>(&predp[(w4 * 16 * Cfg::PT + 16 * t + l15) * 4 + 2 * l4]) = make_float2(pacc[t][0] + pacc[t][1], pacc[t][2] + pacc[t][3]);
        }
        group_barrier();   // B3: partial sums of the projection rows
        if (tid1 < n_em * Cfg::PPW) {
          const int e = tid1 / Cfg::PPW, row = tid1 - e * Cfg::PPW;
          float v = 0.f;
#pragma unroll
          for (int w = 0; w < 4; ++w) v += predp[(w * 16 * Cfg::PT + row) * 4 + e];
          const int s = e == 0 ? es[0] : e == 1 ? es[1] : e == 2 ? es[2] : es[3];
          group_st(px + s * H + prow0 + row, __float_as_uint(v + bpl[row]), stamp, near);
        }
        // ---- off the chain: the recurrent sums of the next step (their partial sums are added behind the next barrier)
#pragma unroll
        for (int t = 0; t < Cfg::LT; ++t) {
          f32x4 racc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int i = 0; i < KS; ++i) racc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(hf[i], wr[t][i], racc, 0, 0, 0);
          if (lane < 32) *reinterpret_cast<float2 *>(&recp[(w4 * NR + 16 * t + l15) * 4 + 2 * l4]) = make_float2(racc[0] + racc[1], racc[2] + racc[3]);
        }
        pend = n_em;
#pragma unroll
        for (int e = 0; e < SL; ++e) pend_slot[e] = es[e];
      } else {
        group_barrier();   // B3
        // ---- exchange 3: this wave's quarter of the new projections
        unsigned long long u[SL][QL];
        const bool got = group_poll(abort_word, gd.spin_limit, [&]() {
#pragma unroll
          for (int e = 0; e < SL; ++e)
            if (e < n_em) {
#pragma unroll
              for (int q = 0; q < QL; ++q) u[e][q] = group_ld(px + es[e] * H + w4 * QK + min(lane + 64 * q, QK - 1));
            }
          bool fresh = true;
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
              if (lane + 64 * q < QK) pfull[es[e] * H + w4 * QK + lane + 64 * q] = __uint_as_float((unsigned)u[e][q]);
          }
      }
    }
    if constexpr (ROLE == 1) load_frames();
    if (rf) {   // slots that took a new utterance: the state after the start token, their first frames
      unsigned long long todo = rf;
      while (todo) {
        const int a = __builtin_amdgcn_readfirstlane(__ffsll((long long)todo) - 1);
        todo &= todo - 1;
        if constexpr (ROLE == 0) {
          for (int i = tid1; i < H; i += 256) pfull[a * H + i] = m.start_p[i];
        } else {
          for (int i = tid1; i < NR; i += 256) recs[a * NR + i] = m.start_rec[unit0 * 4 + i];
          for (int i = tid1; i < Cfg::UPW; i += 256) cst[a * Cfg::UPW + i] = m.start_c[unit0 + i];
        }
      }
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      group_barrier();
    }
  }
  if constexpr (ROLE == 1) {
    if (g == 0 && wave == 7) group_add_counters(c, counts, lane);
  }
}

template <int KS, int CT, int GW, int MODE>
__global__ __launch_bounds__(512) void wind_group_kernel(ModelDev m, CallDev c, GroupDev gd) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem_raw[];
  const int grp = (int)blockIdx.x % kGroups, g = (int)blockIdx.x / kGroups;   // workgroups go to the XCDs in turn
  if (grp >= gd.NG) return;
  if (blockIdx.x == 0 && threadIdx.x == 0) c.stats[kStatLoop] = (unsigned long long)wall_clock64();
  if (threadIdx.x < 256) group_loop<KS, CT, GW, MODE, 0>(m, c, gd, smem_raw, grp, g);
  else group_loop<KS, CT, GW, MODE, 1>(m, c, gd, smem_raw, grp, g);
}

}  // namespace wind
