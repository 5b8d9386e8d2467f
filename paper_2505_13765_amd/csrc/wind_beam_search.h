// Host side of WIND beam search (section "A Novel Beam-search Algorithm for WIND", Algorithm 3):
// the map from frames to hypotheses, recombination, the prefix step, pruning and the expansion
// loop run on the host; every model evaluation (encoder projection, prediction-network steps for
// new label sequences, joiner rows, soft-max, P' of Eq. 1 and the K best pairs) runs on the GPU: on the
// resident workgroups of wind_beam_resident.h where model and search fit them, else in the kernels of wind_beam.h.  Included by wind_api.hip after wind_model and its helpers.
//
// Label sequences are nodes of a trie (parent, label), so that "same sequence" is "same node" and
// "A is a prefix of B" is "A is an ancestor of B".  A node gets a state slot (LSTM h and c of every
// layer, projected output) the first time a hypothesis with that sequence survives pruning; its
// parent always has one by then, because hypotheses are only ever expanded after that point.
#pragma once

namespace {

struct BeamWs {
  float *e, *p, *logits, *lse, *blp, *cl;
  int *cv;
  bf16_t *z, *z_lo;
};

BeamIndex beam_identity() { return BeamIndex{nullptr, 0, {0}}; }
BeamIndex beam_list(const int *device_list) { return BeamIndex{device_list, 0, {0}}; }
BeamIndex beam_inline(const int *host_values, int n) {
  BeamIndex ix{nullptr, n, {0}};
  for (int i = 0; i < n; ++i) ix.inl[i] = host_values[i];
  return ix;
}

// Lays the scoring workspace for up to n frames, Bh hypotheses and `rows` joiner rows out from `base`
// (null: sizes only) and returns its size in bytes.
size_t beam_carve(const wind_model *m, size_t n, size_t Bh, size_t rows, char *base, BeamWs *ws) {
  const ModelDev &d = m->dev;
  const size_t rows_pad = round_up(rows, JointCfg::BM), V1 = (size_t)d.V + 1;
  size_t off = 0;
  auto take = [&](size_t bytes) { size_t o = off; off += round_up(bytes, 256); return o; };
  const size_t o_e = take(n * d.Hj * 4), o_p = take(Bh * d.Hj * 4);
  const size_t o_z = take(rows_pad * d.Hj * 2), o_zlo = take(rows_pad * d.Hj * 2), o_lg = take(rows * V1 * 4);
  const size_t o_lse = take(rows * 4), o_blp = take(rows * 4), o_cl = take(rows * kBeamMaxK * 4), o_cv = take(rows * kBeamMaxK * 4);
  if (base && ws) {
    ws->e = (float *)(base + o_e); ws->p = (float *)(base + o_p); ws->logits = (float *)(base + o_lg);
    ws->z = (bf16_t *)(base + o_z);
    ws->z_lo = (bf16_t *)(base + o_zlo);
    ws->lse = (float *)(base + o_lse); ws->blp = (float *)(base + o_blp); ws->cl = (float *)(base + o_cl);
    ws->cv = (int *)(base + o_cv);
  }
  return off;
}

// The model's own scoring workspace, allocated on first use and regrown on demand.
int beam_workspace_reserve(wind_model *m, size_t off, hipStream_t s) {
  if (off > m->beam_ws_bytes) {
    HIP_TRY(hipDeviceSynchronize());
    if (m->beam_ws) HIP_TRY(hipFree(m->beam_ws));
    m->beam_ws = nullptr;
    m->beam_ws_bytes = 0;
    HIP_TRY(hipMalloc(&m->beam_ws, off));
    m->beam_ws_bytes = off;
    HIP_TRY(hipMemsetAsync(m->beam_ws, 0, off, s));   // the MFMA pass reads whole row tiles; on the stream that the pass runs on
  }
  return WIND_OK;
}
int beam_workspace(wind_model *m, size_t n, size_t Bh, size_t rows, BeamWs *ws, hipStream_t s) {
  const int rc = beam_workspace_reserve(m, beam_carve(m, n, Bh, rows, nullptr, nullptr), s);
  if (rc) return rc;
  beam_carve(m, n, Bh, rows, (char *)m->beam_ws, ws);
  return WIND_OK;
}

// logits[(b, t), :] = joiner row of frame t of e_win ([n, Hj] projected frames) and hypothesis b (row
// pi(b) of p).  bf16 models: the MFMA pass on the hidden vector rounded to bf16, or, with option
// "beam_exact", on its split into two bf16 vectors (close to fp32 accuracy).  fp32 models: fp32 FMA.
void beam_enqueue_logits(wind_model *m, const BeamWs &ws, const float *e_win, int n, const float *p, const BeamIndex &pi,
                         int Bh, hipStream_t s) {
  const ModelDev &d = m->dev;
  const size_t rows = (size_t)Bh * n, rows_pad = round_up(rows, JointCfg::BM), V1 = (size_t)d.V + 1;
  const size_t tiny_tiles = ((V1 + 31) / 32) * ((rows + 31) / 32), row_tiles = (rows + PredCfg::BM - 1) / PredCfg::BM,
               col_tiles = (V1 + PredCfg::BN - 1) / PredCfg::BN;
  // 32 x 32 blocks, which form their hidden rows themselves, while they fit the chip one per CU: every column tile forms all rows again.  Whole scoring step, us,
  // 32 x 32 / 64 x 64 blocks: 8192 labels, 1024 units (264 blocks per 32 rows), 16 rows 65 / 62, 64 71 / 64, 128 84 / 67, 256 109 / 76; 1024 labels, 640 units
  // (33), 32 rows 48 / 52, 64 49 / 52, 256 54.5 / 53.7.  64 x 64 blocks up to eight per CU, 128 x 128 above: 1024 labels, 512 rows 57 / 67, 1024 rows 62 / 70;
  // 8192 labels, 512 rows 90 / 91, 1024 113 / 115, 4096 265 / 232.
  if (m->dtype == WIND_BF16 && d.Hj <= kBeamTinyMaxHj && rows <= (size_t)kBeamTinyMaxRows && tiny_tiles <= (size_t)m->cu_count) {
    const int split = m->opt_beam_exact ? 1 : 0;
    const size_t smem = beam_tiny_smem(d.Hj, split);
    const dim3 grid((unsigned)round_up((V1 + 31) / 32, 8), (unsigned)((rows + 31) / 32));
    auto go = [&](auto kernel) { kernel<<<grid, 512, smem, s>>>(d, e_win, p, pi, n, (int)rows, split, ws.logits); };
    if (d.Hj <= 256) go(beam_logits_tiny_kernel<1>);
    else if (d.Hj <= 512) go(beam_logits_tiny_kernel<2>);
    else if (d.Hj <= 768) go(beam_logits_tiny_kernel<3>);
    else go(beam_logits_tiny_kernel<4>);
  } else if (m->dtype == WIND_BF16) {
    bf16_t *z_lo = m->opt_beam_exact ? ws.z_lo : nullptr;
    beam_hidden_kernel<<<(unsigned)rows, 256, 0, s>>>(e_win, p, pi, ws.z, z_lo, n, d.Hj);
    if (row_tiles * col_tiles <= 8 * (size_t)m->cu_count) {
      const dim3 grid((unsigned)round_up(col_tiles, 8), (unsigned)row_tiles);
      beam_logits_dma_kernel<PredCfg><<<grid, PredCfg::NT, PredCfg::SMEM_BYTES, s>>>(d, ws.z, z_lo, (int)rows, ws.logits);
    } else {
      dim3 grid((unsigned)(rows_pad / JointCfg::BM), (unsigned)((V1 + JointCfg::BN - 1) / JointCfg::BN));
      joint_mfma_store_kernel<JointCfg><<<grid, JointCfg::NT, JointCfg::SMEM_BYTES, s>>>(d, ws.z, z_lo, (int)rows, ws.logits);
    }
  } else {
    beam_logits_kernel<float><<<(unsigned)rows, 256, (size_t)d.Hj * 4, s>>>(d, e_win, p, pi, n, ws.logits);
  }
}

// The K best (label, jump) pairs of every hypothesis from its n rows of logits.
void beam_enqueue_topk(wind_model *m, const BeamWs &ws, int n, int Bh, int K, int32_t *out_labels, int32_t *out_jumps,
                       float *out_scores, hipStream_t s) {
  const ModelDev &d = m->dev;
  const size_t rows = (size_t)Bh * n, V1 = (size_t)d.V + 1;
  if (V1 <= 256 * 36) {
    // one workgroup per row, then one wave per hypothesis
    if (V1 <= 256 * 8) beam_row_kernel<8, 4><<<(unsigned)rows, 256, 0, s>>>(ws.logits, d.V, K, ws.lse, ws.blp, ws.cl, ws.cv);
    else beam_row_kernel<18, 8><<<(unsigned)rows, 512, 0, s>>>(ws.logits, d.V, K, ws.lse, ws.blp, ws.cl, ws.cv);
    beam_merge_kernel<<<(unsigned)Bh, 64, 0, s>>>(ws.lse, ws.blp, ws.cl, ws.cv, n, d.V, K, out_labels, out_jumps, out_scores);
  } else if (K <= 8) {
    beam_score_kernel<8><<<(unsigned)Bh, 256, 0, s>>>(ws.logits, n, d.V, K, out_labels, out_jumps, out_scores);
  } else if (K <= 16) {
    beam_score_kernel<16><<<(unsigned)Bh, 256, 0, s>>>(ws.logits, n, d.V, K, out_labels, out_jumps, out_scores);
  } else {
    beam_score_kernel<32><<<(unsigned)Bh, 256, 0, s>>>(ws.logits, n, d.V, K, out_labels, out_jumps, out_scores);
  }
}

// out[r, :] = w x[r] + bias for fp32 rows x, weights in the model's storage type: the encoder projection of `n` frames to `e` and, with
// rows, the prediction network's projection of `rows` hidden vectors to `p`, in one launch.
void beam_enqueue_projections(wind_model *m, const float *frames, float *e, int n, const float *hidden, float *p, int rows, hipStream_t s) {
  constexpr int kR = 8;   // rows that share one pass over a weight row
  const ModelDev &d = m->dev;
  const int jb = (d.Hj + 3) / 4, blocks_e = jb * ((n + kR - 1) / kR), blocks_p = jb * ((rows + kR - 1) / kR);
  const BeamLinear le{d.w_enc, d.b_enc, frames, e, n, d.Hj, d.D, m->dtype == WIND_BF16}, lp{d.w_pred, d.b_pred, hidden, p, rows, d.Hj, d.Hp, 0};
  if (m->dtype == WIND_BF16) beam_linear_kernel<bf16_t, kR><<<(unsigned)(blocks_e + blocks_p), 256, 0, s>>>(le, lp, blocks_e);
  else beam_linear_kernel<float, kR><<<(unsigned)(blocks_e + blocks_p), 256, 0, s>>>(le, lp, blocks_e);
}

// ---- state pool and staging ---------------------------------------------------------------------
constexpr int kBeamCompRows = 1024;   // completion rows (prefix step) evaluated per batch
constexpr int kBeamStageInts = 2 * kBeamCompRows;   // device lists of a large completion batch: slots, labels
constexpr int kBeamResScores = 0, kBeamResLabels = kBeamMaxK * kBeamMaxK, kBeamResJumps = 2 * kBeamMaxK * kBeamMaxK,
              kBeamResComp = 3 * kBeamMaxK * kBeamMaxK, kBeamResWords = 3 * kBeamMaxK * kBeamMaxK + kBeamCompRows;

int beam_pool_reserve(wind_model *m, int slots, hipStream_t s) {
  BeamPool &bp = m->beam_pool;
  const ModelDev &d = m->dev;
  if (!bp.h_stage) {
    // results land in pinned host memory that the kernels write directly: a pass ends with a stream
    // synchronisation and no copy
    HIP_TRY(hipHostMalloc((void **)&bp.h_stage, sizeof(int) * kBeamStageInts, hipHostMallocDefault));
    HIP_TRY(hipHostMalloc((void **)&bp.h_res, 4 * kBeamResWords, hipHostMallocDefault));
    HIP_TRY(hipMalloc((void **)&bp.d_stage, sizeof(int) * kBeamStageInts));
    HIP_TRY(hipHostGetDevicePointer(&bp.d_res, bp.h_res, 0));
  }
  if (slots <= bp.cap) return WIND_OK;
  int cap = bp.cap ? bp.cap : 1024;
  while (cap < slots) cap *= 2;
  const size_t st = (size_t)d.L * d.Hp;
  float *h = nullptr, *c = nullptr, *p = nullptr;
  HIP_TRY(hipMalloc((void **)&h, (size_t)cap * st * 4));
  HIP_TRY(hipMalloc((void **)&c, (size_t)cap * st * 4));
  HIP_TRY(hipMalloc((void **)&p, (size_t)cap * d.Hj * 4));
  if (bp.cap) {
    HIP_TRY(hipMemcpyAsync(h, bp.h, (size_t)bp.cap * st * 4, hipMemcpyDeviceToDevice, s));
    HIP_TRY(hipMemcpyAsync(c, bp.c, (size_t)bp.cap * st * 4, hipMemcpyDeviceToDevice, s));
    HIP_TRY(hipMemcpyAsync(p, bp.p, (size_t)bp.cap * d.Hj * 4, hipMemcpyDeviceToDevice, s));
    HIP_TRY(hipStreamSynchronize(s));
    (void)hipFree(bp.h); (void)hipFree(bp.c); (void)hipFree(bp.p);
  }
  bp.h = h; bp.c = c; bp.p = p; bp.cap = cap;
  return WIND_OK;
}

void beam_pool_free(wind_model *m) {
  BeamPool &bp = m->beam_pool;
  if (bp.h) (void)hipFree(bp.h);
  if (bp.c) (void)hipFree(bp.c);
  if (bp.p) (void)hipFree(bp.p);
  if (bp.e_all) (void)hipFree(bp.e_all);
  if (bp.d_stage) (void)hipFree(bp.d_stage);
  if (bp.h_stage) (void)hipHostFree(bp.h_stage);
  if (bp.h_res) (void)hipHostFree(bp.h_res);
  bp = BeamPool{};
}

// One prediction-network step for `rows` (at most 32) new label sequences.
void beam_enqueue_decoder_step(wind_model *m, int rows, const int *parent, const int *child, const int *tok, hipStream_t s) {
  const ModelDev &d = m->dev;
  BeamPool &bp = m->beam_pool;
  const BeamIndex pa = beam_inline(parent, rows), ch = beam_inline(child, rows), tk = beam_inline(tok, rows);
  constexpr int R = 4;
  const unsigned lb = (unsigned)((d.Hp + 3) / 4), pb = (unsigned)((d.Hj + 3) / 4);
  for (int l = 0; l < d.L; ++l) {
    if (m->dtype == WIND_BF16) beam_lstm_layer_kernel<bf16_t, R><<<lb, 256, 0, s>>>(d, bp.h, bp.c, l, rows, pa, ch, tk);
    else beam_lstm_layer_kernel<float, R><<<lb, 256, 0, s>>>(d, bp.h, bp.c, l, rows, pa, ch, tk);
  }
  if (m->dtype == WIND_BF16) beam_pred_kernel<bf16_t, R><<<pb, 256, 0, s>>>(d, bp.h, bp.p, rows, ch);
  else beam_pred_kernel<float, R><<<pb, 256, 0, s>>>(d, bp.h, bp.p, rows, ch);
}

// ---- resident workgroups
struct BeamInstance {
  void (*search)(ModelDev, BeamResDev);
  void (*scores)(ModelDev, BeamResDev);
  void (*phases[4])(ModelDev, BeamResDev);
  size_t smem, smem_rows;
};
template <int KS>
constexpr BeamInstance beam_instance() { return {beam_search_kernel<KS>,
                                                                   beam_scores_kernel<KS>,
                                                                   {beam_scores_phase_kernel<KS, 0>, beam_scores_phase_kernel<KS, 1>, beam_scores_phase_kernel<KS, 2>, beam_scores_phase_kernel<KS, 3>},
                                                                   BeamResCfg<KS>::smem, BeamResCfg<KS>::smem_rows}; }
const BeamInstance kBeamInstances[] = {beam_instance<1>(), beam_instance<2>(), beam_instance<3>(), beam_instance<4>(), beam_instance<5>()};   // by width / 128
// Models that resident workgroups hold: bf16, one LSTM layer as wide as the joiner and of up to 640 units, up to 1024 labels, as the
// resident groups of the decoder; and the options that ask for those
bool beam_resident_model(const wind_model *m) {
  const ModelDev &d = m->dev;
  return m->dtype == WIND_BF16 && d.start_p && d.V <= kGroupMaxV && d.Hj <= 640 && m->cu_count >= kGroups * 32 && m->device >= 0 && m->device < kMaxDevices && m->opt_loop_kernel &&
         m->opt_loop_fused && m->opt_loop_one_xcd && !m->opt_profile && m->opt_graph && !m->opt_host_sync && !m->opt_debug_stamps;
}
int beam_resident_reserve(wind_model *m, hipStream_t s) {
  BeamResident &br = m->beam_res;
  if (!br.mem || br.seq > 0xF0000000u || br.session > 0x0F000000u) {   // numbers that no word in the buffers has
    HIP_TRY(hipDeviceSynchronize());
    if (!br.mem) HIP_TRY(hipMalloc((void **)&br.mem, sizeof(BeamGroupMem) * kGroups));
    HIP_TRY(hipMemsetAsync(br.mem, 0, sizeof(BeamGroupMem) * kGroups, s));
    br.seq = br.session = br.written = 0;
  }
  if (!br.host) {
    HIP_TRY(hipHostMalloc((void **)&br.host, sizeof(BeamResident::Host), hipHostMallocCoherent));
    std::memset(br.host, 0, sizeof(BeamResident::Host));
    HIP_TRY(hipHostGetDevicePointer((void **)&br.dev, br.host, 0));
  }
  return WIND_OK;
}

constexpr unsigned kBeamSessionCommands = 256;    // commands of one launch: whatever else waits for the stream gets its turn
constexpr int kBeamRestSearches = 8;              // searches on launches after one whose workgroups could not meet
constexpr double kBeamIdleMs = 1.0;               // without a command for this long the workgroups leave
// .. of a search with a callback, which may take any time and may wait for the GPU, workgroups included: about a pass with launches.  Once they have
// left for that reason kBeamSlowCallbacks times in a row they are sent away ahead of the search's callbacks.  A callback that synchronises with the device, 280 passes: 16.2 ms
// on launches, 292 with a wait of 1 ms each, now 12
constexpr double kBeamCallbackIdleMs = 0.04;
constexpr int kBeamSlowCallbacks = 3;

// The resident workgroups as one search uses them.  They stay from open() to close(), or until they have been idle, have
// had their number of commands, or another call waits for its turn; the next command launches them again.
struct BeamSession {
  wind_model *m;
  hipStream_t s;
  bool usable = false, is_open = false;   // usable: shape and options allow it, and nothing has gone wrong so far
  bool callback = false;
  int idle_callbacks = 0;   // callbacks in a row in which the workgroups went idle; from kBeamSlowCallbacks on for the rest of the search
  unsigned long long turn = 0;
  unsigned commands = 0;

  BeamSession(wind_model *m_, hipStream_t s_) : m(m_), s(s_) {}
  ~BeamSession() { close(); }
  BeamSession(const BeamSession &) = delete;
  BeamSession &operator=(const BeamSession &) = delete;

  int open() {
    BeamResident &br = m->beam_res;
    BeamPool &bp = m->beam_pool;
    ResidentGate &gate = g_resident[m->device];
    BeamResDev r{};
    r.host_cmd = br.dev->cmd; r.host_res = br.dev->res; r.host_exit = &br.dev->exit;
    r.mem = br.mem;
    r.h = bp.h; r.c = bp.c; r.p = bp.p; r.e_all = bp.e_all;
    r.session = ++br.session;
    r.first = br.seq;
    r.spin_limit = (unsigned)m->opt_loop_spin_limit;
    r.start_limit = std::min(r.spin_limit, kGroupStartPolls);
    r.idle_ticks = (unsigned long long)((callback ? kBeamCallbackIdleMs : kBeamIdleMs) * m->clock_khz);
    std::lock_guard<std::mutex> lock(gate.mutex);
    int rc = resident_enter(gate, s);
    if (rc) return rc;
    const BeamInstance &k = kBeamInstances[m->dev.Hj / 128 - 1];
    k.search<<<kGroups * kBeamResWgs, 512, k.smem, s>>>(m->dev, r);
    rc = check_launch("beam search on resident workgroups");
    if (rc) return rc;
    is_open = true;   // also if the event fails: the kernel is there
    ++m->route.beam_launches;
    commands = 0;
    return resident_leave(gate, s, &turn);
  }
  void post(const unsigned (&words)[kBeamCmdWords]) {
    BeamResident &br = m->beam_res;
    for (int i = 0; i < kBeamCmdWords; ++i)
      __atomic_store_n(&br.host->cmd[i], (unsigned long long)words[i] | ((unsigned long long)br.seq << 32), __ATOMIC_RELAXED);
  }
  // Sends everybody away; they leave within microseconds, and whoever waits for this stream or for its turn goes on behind them
  void close() {
    if (!is_open) return;
    const unsigned quit[kBeamCmdWords] = {kBeamCmdQuit};
    ++m->beam_res.seq;
    post(quit);
    is_open = false;
  }
  // One command: true in `done` once `arrived` says that all its results are in pinned memory.  Not done: the workgroups could not
  // meet or gave up, nothing of them runs any more, and the caller takes the launches from here on.
  template <class Arrived>
  int run(const unsigned (&words)[kBeamCmdWords], int nres, const Arrived &arrived, bool *done) {
    BeamResident &br = m->beam_res;
    *done = false;
    if (is_open && (commands >= kBeamSessionCommands || g_resident[m->device].turn.load(std::memory_order_relaxed) != turn)) close();
    bool stayed = is_open;
    for (;;) {
      ++br.seq;   // a number of its own for every try: under the last one idle workgroups have been told to leave
      for (int i = 0; i < nres; ++i) __atomic_store_n(&br.host->res[i], 0ull, __ATOMIC_RELAXED);
      post(words);
      if (!is_open) {
        const int rc = open();
        if (rc) return rc;
      }
      ++commands;
      bool left = false;
      for (unsigned spins = 1; !left; ++spins) {
        if (arrived()) {
          *done = true;
          ++m->route.beam_commands;
          if (stayed && idle_callbacks < kBeamSlowCallbacks) idle_callbacks = 0;
          return WIND_OK;
        }
        left = __atomic_load_n(&br.host->exit, __ATOMIC_ACQUIRE) >> 2 == br.session;
        if (!left && (spins & 0x3FFFu) == 0) {   // a kernel that failed never says that it has left
          const hipError_t e = hipStreamQuery(s);
          if (e != hipSuccess && e != hipErrorNotReady) return fail(WIND_ERR_HIP, std::string("beam search: ") + hipGetErrorString(e));
          left = e == hipSuccess;
        }
        __builtin_ia32_pause();
      }
      is_open = false;
      HIP_TRY(hipStreamSynchronize(s));
      if (arrived()) { *done = true; ++m->route.beam_commands; return WIND_OK; }
      if (__atomic_load_n(&br.host->exit, __ATOMIC_ACQUIRE) != (br.session << 2 | kBeamExitIdle)) {
        usable = false;
        br.rest_searches = kBeamRestSearches;   // the wait for the workgroups took up to 12 ms: the next searches do without
        ++m->route.beam_gave_up;
        return WIND_OK;
      }
      ++m->route.beam_idle;
      stayed = false;
      if (callback) ++idle_callbacks;
      // idle when the command came: the next launch takes it
    }
  }
};

// Scoring steps that the resident workgroups' kernel computes: the loads are 16 bytes wide
bool beam_scores_shape(const wind_model *m, const float *enc_window, int n, const float *dec_out, int Bh, int K) {
  return Bh <= kGroups * kBeamResHyps && n <= kBeamResFrames && K <= kBeamResHyps && beam_resident_model(m) && ((uintptr_t)enc_window | (uintptr_t)dec_out) % 16 == 0;
}

// The same sums in launches that wait for nobody (see BeamRes::score), in `area`.  Static entry point, n = 16, K = 8, 640 units, 1024 labels, called
// alone: 1 / 8 / 16 / 64 hypotheses 41 / 41 / 42 / 53 us; as two projections, logits, rows and merge 53 / 48 / 52 / 73
int beam_scores_phases(wind_model *m, const BeamPhaseArea &area, const float *enc_window, int n, const float *dec_out, int Bh, int K, int32_t *out_labels,
                       int32_t *out_jumps, float *out_scores, hipStream_t s) {
  BeamResDev r{};
  r.mem = reinterpret_cast<BeamGroupMem *>(area.base);   // not looked at
  r.area = area;
  r.session = r.first = 1;
  r.enc = enc_window; r.dec = dec_out;
  r.n = n; r.Bh = Bh; r.K = K; r.split = m->opt_beam_exact ? 1 : 0;
  r.out_labels = out_labels; r.out_jumps = out_jumps; r.out_scores = out_scores;
  const BeamInstance &k = kBeamInstances[m->dev.Hj / 128 - 1];
  const int hyps = (Bh + kGroups - 1) / kGroups;
  const int wgs[4] = {kBeamResWgs, kBeamResWgs, std::min(kBeamResWgs, hyps * n), hyps};   // workgroups that have a part in a phase
  for (int p = 0; p < 4; ++p) k.phases[p]<<<kGroups * wgs[p], 512, p < 2 ? k.smem : k.smem_rows, s>>>(m->dev, r);
  return check_launch("beam scoring step");
}

// Workgroups of a scoring step wait this long (about 1.5 ms) for all of their group to be on the chip: beside a stream of large matrix products a step
// takes 0.95 ms that way and 3.5 as several launches, which each wait for CUs as well.  Where something keeps CUs for longer, every step would
// lose that: after a failure the next kBeamRest steps take the launches at once.
constexpr unsigned kBeamStepStartPolls = 1u << 13;
constexpr int kBeamRest = 256;

// One scoring step of a shape that beam_scores_shape takes, as a single launch, or, if its workgroups cannot meet, as several.  Either way the same
// sums, to the bit; returns with the results in the caller's buffers.
int beam_scores_groups(wind_model *m, const float *enc_window, int n, const float *dec_out, int Bh, int K, int32_t *out_labels,
                       int32_t *out_jumps, float *out_scores, hipStream_t s) {
  BeamResident &br = m->beam_res;
  if (br.rest_steps > 0) {
    --br.rest_steps;
  } else {
    int rc = beam_resident_reserve(m, s);
    if (rc) return rc;
    BeamResDev r{};
    r.host_exit = &br.dev->exit;
    r.mem = br.mem;
    r.session = ++br.session;
    r.first = ++br.seq;
    r.spin_limit = (unsigned)m->opt_loop_spin_limit;
    r.start_limit = std::min(r.spin_limit, kBeamStepStartPolls);
    r.enc = enc_window; r.dec = dec_out;
    r.n = n; r.Bh = Bh; r.K = K; r.split = m->opt_beam_exact ? 1 : 0;
    r.out_labels = out_labels; r.out_jumps = out_jumps; r.out_scores = out_scores;
    r.written = br.written += (unsigned)Bh;
    ResidentGate &gate = g_resident[m->device];
    unsigned long long turn = 0;
    {
      std::lock_guard<std::mutex> lock(gate.mutex);
      rc = resident_enter(gate, s);
      if (rc) return rc;
      const BeamInstance &k = kBeamInstances[m->dev.Hj / 128 - 1];
      k.scores<<<kGroups * kBeamResWgs, 512, k.smem, s>>>(m->dev, r);
      rc = check_launch("beam scoring step");
      if (rc) return rc;
      rc = resident_leave(gate, s, &turn);
      if (rc) return rc;
    }
    bool done = false;
    const auto arrived = [&]() { return __atomic_load_n(&br.host->exit, __ATOMIC_ACQUIRE) >> 2 == r.session; };
    for (unsigned spins = 1; !(done = arrived()); ++spins) {
      if ((spins & 0x3FFu) == 0) {
        const hipError_t e = hipStreamQuery(s);
        if (e != hipSuccess && e != hipErrorNotReady) return fail(WIND_ERR_HIP, std::string("beam scoring step: ") + hipGetErrorString(e));
        if (e == hipSuccess) {
          done = arrived();
          break;
        }
      }
      __builtin_ia32_pause();
    }
    resident_done(gate, turn);
    ++(done ? m->route.scores_resident : m->route.scores_gave_up);
    if (done) return WIND_OK;
    br.rest_steps = kBeamRest;
    HIP_TRY(hipMemsetAsync(&br.mem[0].word[1], 0, sizeof(unsigned), s));   // some of its hypotheses may have been written: the count starts again
    br.written = 0;
  }
  BeamPhaseArea area = beam_phase_area(nullptr, m->dev.Hj, m->dev.V, n, Bh, K);
  int rc = beam_workspace_reserve(m, (size_t)area.bytes * std::min(Bh, kGroups), s);
  if (rc) return rc;
  area.base = (unsigned char *)m->beam_ws;
  rc = beam_scores_phases(m, area, enc_window, n, dec_out, Bh, K, out_labels, out_jumps, out_scores, s);
  if (rc) return rc;
  HIP_TRY(hipStreamSynchronize(s));
  return WIND_OK;
}

struct BeamNode {
  int parent, token, depth, slot;
};
struct BeamHyp {
  int node;
  double score;
  int sym;      // labels already placed on the frame the hypothesis rests on
  int stamps;   // time stamps of its labels: the last one's entry in a list of (frame, entry before), -1: no labels
};
struct BeamStamp {
  int frame, before;
};

// (node, label) -> child node: open addressing, a power of two of places, at most half of them taken
struct BeamChildren {
  std::vector<std::pair<unsigned long long, int>> place{(size_t)1 << 12, {0ull, -1}};
  size_t taken = 0;
  // the child's node, or a place that holds -1 and that the caller fills
  int &find(int parent, int token) {
    if (2 * (taken + 1) > place.size()) {
      std::vector<std::pair<unsigned long long, int>> old(place.size() * 2, {0ull, -1});
      old.swap(place);
      for (const auto &o : old)
        if (o.second >= 0) at(o.first) = o;
    }
    const unsigned long long key = ((unsigned long long)(unsigned)parent << 32) | (unsigned)token;
    auto &p = at(key);
    p.first = key;
    if (p.second < 0) ++taken;
    return p.second;
  }
  std::pair<unsigned long long, int> &at(unsigned long long key) {
    size_t i = (size_t)((key * 0x9E3779B97F4A7C15ull) >> 32) & (place.size() - 1);
    while (place[i].second >= 0 && place[i].first != key) i = (i + 1) & (place.size() - 1);
    return place[i];
  }
};

double beam_logaddexp(double a, double b) {
  if (a == -INFINITY) return b;
  if (b == -INFINITY) return a;
  const double mx = a > b ? a : b;
  return mx + std::log(std::exp(a - mx) + std::exp(b - mx));
}

int beam_decode(wind_model *m, const float *enc_out, int T, int window, int K, int S, int prefix_mode, int32_t *out_tokens,
                int32_t *out_frames, int cap, int32_t *out_count, double *out_score, wind_beam_stats *stats,
                wind_beam_round_fn on_round, void *user, void *stream) {
  if (!m || (!enc_out && T > 0) || !out_tokens || !out_frames || !out_count || !out_score)
    return fail(WIND_ERR_ARG, "null argument");
  if (T < 0 || cap < 0) return fail(WIND_ERR_ARG, "T and cap must not be negative");
  if (window < 1 || window > kBeamMaxWindow) return fail(WIND_ERR_ARG, "window must have 1..64 frames");
  if (K < 1 || K > kBeamMaxK) return fail(WIND_ERR_ARG, "K must be in 1..32");
  if (S < 1) return fail(WIND_ERR_ARG, "S must be at least 1");
  if (prefix_mode < WIND_PREFIX_OFF || prefix_mode > WIND_PREFIX_REMOVE) return fail(WIND_ERR_ARG, "unknown prefix mode");
  wind_beam_stats st{};
  *out_count = 0;
  *out_score = 0.0;
  if (stats) *stats = st;
  if (T == 0) return WIND_OK;

  const ModelDev &d = m->dev;
  hipStream_t s = (hipStream_t)stream;
  BeamPool &bp = m->beam_pool;
  const int V = d.V, V1 = V + 1;
  BeamWs ws;
  int rc = beam_workspace(m, (size_t)window, (size_t)kBeamMaxK, (size_t)std::max(kBeamMaxK * window, kBeamCompRows), &ws, s);
  if (rc) return rc;
  rc = beam_pool_reserve(m, 1024, s);
  if (rc) return rc;
  // every frame through the encoder projection, once
  if ((size_t)T * d.Hj * 4 > bp.e_bytes) {
    HIP_TRY(hipStreamSynchronize(s));
    if (bp.e_all) (void)hipFree(bp.e_all);
    bp.e_all = nullptr; bp.e_bytes = 0;
    HIP_TRY(hipMalloc((void **)&bp.e_all, (size_t)T * d.Hj * 4));
    bp.e_bytes = (size_t)T * d.Hj * 4;
  }
  beam_enqueue_projections(m, enc_out, bp.e_all, T, nullptr, nullptr, 0, s);

  // trie of label sequences; slot 0 holds the zero state, the empty sequence is one step from it on the start id
  std::vector<BeamNode> nodes;
  BeamChildren children;
  std::vector<BeamStamp> stamps;
  int next_slot = 2;
  nodes.push_back(BeamNode{-1, V, 0, 1});
  const size_t slot_sz = (size_t)d.L * d.Hp;
  HIP_TRY(hipMemsetAsync(bp.h, 0, slot_sz * 4, s));
  HIP_TRY(hipMemsetAsync(bp.c, 0, slot_sz * 4, s));
  {
    const int zero_slot = 0, root_slot = 1, start_id = V;
    beam_enqueue_decoder_step(m, 1, &zero_slot, &root_slot, &start_id, s);
  }
  rc = check_launch("beam search set-up");
  if (rc) return rc;
  st.decoder_steps = 1;
  BeamSession session(m, s);
  BeamResident &br = m->beam_res;
  if (K <= kBeamResHyps && window <= kBeamResFrames && beam_resident_model(m)) {
    rc = beam_resident_reserve(m, s);
    if (rc) return rc;
    if (br.rest_searches > 0) --br.rest_searches;
    else session.usable = true;
    session.callback = on_round != nullptr;
  }
  auto put = [](unsigned (&words)[kBeamCmdWords], int kind, int fresh, int Bh, int n, int t, int K, int split) {
    words[kBeamAtHead] = (unsigned)(kind | fresh << 8 | Bh << 16 | n << 24);
    words[kBeamAtFrame] = (unsigned)t;
    words[kBeamAtK] = (unsigned)(K | split << 8);
  };

  auto tokens_of = [&](int node) {
    std::vector<int> t((size_t)nodes[node].depth);
    for (int q = node; nodes[q].parent >= 0; q = nodes[q].parent) t[(size_t)nodes[q].depth - 1] = nodes[q].token;
    return t;
  };
  auto child_node = [&](int parent, int token) {
    int &child = children.find(parent, token);
    if (child < 0) {
      child = (int)nodes.size();
      nodes.push_back(BeamNode{parent, token, nodes[parent].depth + 1, -1});
    }
    return child;
  };
  auto frames_of = [&](const BeamHyp &h) {
    std::vector<int> f((size_t)nodes[h.node].depth);
    size_t i = f.size();
    for (int q = h.stamps; q >= 0; q = stamps[q].before) f[--i] = stamps[q].frame;
    return f;
  };
  // what a pass knows about a node: valid if its pass is the present one
  struct Mark {
    int64_t pass;
    int value;
  };
  std::vector<Mark> hyp_at, row_at;
  auto mark = [&](std::vector<Mark> &marks, int64_t pass, int node) -> int * {   // the node's value in this pass, or null
    if ((size_t)node < marks.size() && marks[node].pass == pass) return &marks[node].value;
    return nullptr;
  };
  auto set_mark = [&](std::vector<Mark> &marks, int64_t pass, int node, int value) {
    if ((size_t)node >= marks.size()) marks.resize(nodes.size() + nodes.size() / 2 + 64, Mark{-1, 0});
    marks[node] = Mark{pass, value};
  };
  // step 1: one entry per label sequence, probabilities added in list order; the time stamps and
  // label count of the most probable duplicate are kept (ties: smaller time stamps, then count)
  int64_t look = 0;
  std::vector<BeamHyp> merged;
  std::vector<double> best_single;
  auto recombine = [&](std::vector<BeamHyp> &hyps) {
    ++look;
    merged.clear();
    best_single.clear();
    for (const BeamHyp &h : hyps) {
      const int *at = mark(hyp_at, look, h.node);
      if (!at) {
        set_mark(hyp_at, look, h.node, (int)merged.size());
        best_single.push_back(h.score);
        merged.push_back(h);
        continue;
      }
      BeamHyp &g = merged[*at];
      double &bs = best_single[*at];
      const double total = beam_logaddexp(g.score, h.score);
      bool take = h.score > bs;
      if (h.score == bs) {
        const std::vector<int> fh = frames_of(h), fg = frames_of(g);
        take = fh < fg || (fh == fg && h.sym < g.sym);
      }
      if (take) { g.stamps = h.stamps; g.sym = h.sym; bs = h.score; }
      g.score = total;
    }
    hyps.swap(merged);
  };

  std::vector<std::vector<BeamHyp>> resting((size_t)T + 1);   // by frame; T: finished
  resting[0].push_back(BeamHyp{0, 0.0, 0, -1});
  std::vector<BeamHyp> hyps, kept;
  std::vector<int> order;
  std::vector<int> cb_len, cb_tok, cb_fr, cb_sym;
  std::vector<double> cb_score;
  for (int t = 0; t < T;) {
    if (resting[t].empty()) {
      std::vector<BeamHyp>().swap(resting[t]);
      ++t;
      continue;
    }
    hyps.clear();
    hyps.swap(resting[t]);   // new ones may come to rest on the same frame: the next pass
    ++st.rounds;
    st.max_pending = std::max<int64_t>(st.max_pending, (int64_t)hyps.size());
    recombine(hyps);

    // step 2: every B receives, from each proper prefix A in the set, A's probability (as it was
    // before this step) times the probability of emitting the missing labels on frame t
    if (prefix_mode != WIND_PREFIX_OFF && hyps.size() > 1) {
      struct Pair { size_t a, b; };
      std::vector<Pair> pairs;
      std::vector<int> row_node;   // child nodes X by row, which holds log P(label(X) | t, decoder(parent(X))); row_at: the row of a node
      for (size_t b = 0; b < hyps.size(); ++b) {
        int q = hyps[b].node;
        for (int up = 1; up < S && nodes[q].parent >= 0; ++up) {
          q = nodes[q].parent;
          const int *at = mark(hyp_at, look, q);   // recombine's: every hypothesis has its place there
          if (!at || hyps[*at].sym + up >= S) continue;
          pairs.push_back(Pair{(size_t)*at, b});
          for (int x = hyps[b].node; x != q; x = nodes[x].parent)
            if (!mark(row_at, look, x)) {
              set_mark(row_at, look, x, (int)row_node.size());
              row_node.push_back(x);
            }
        }
      }
      if (!pairs.empty()) {
        std::vector<float> lp(row_node.size());
        size_t r_done = 0;
        while (session.usable && r_done < row_node.size()) {
          const int rows = (int)std::min<size_t>(kBeamPrefixRows, row_node.size() - r_done);
          unsigned words[kBeamCmdWords] = {0};
          put(words, kBeamCmdComplete, 0, rows, 1, t, K, m->opt_beam_exact ? 1 : 0);
          for (int r = 0; r < rows; ++r) {
            const BeamNode &x = nodes[row_node[r_done + r]];
            words[kBeamAtHyp + r] = (unsigned)nodes[x.parent].slot;
            words[kBeamAtRowTok + r] = (unsigned)x.token;
          }
          bool done = false;
          rc = session.run(words, rows, [&]() {
            for (int r = 0; r < rows; ++r)
              if (__atomic_load_n(&br.host->res[r], __ATOMIC_RELAXED) >> 32 != (br.seq | 0x80000000u)) return false;
            return true;
          }, &done);
          if (rc) return rc;
          if (!done) break;
          for (int r = 0; r < rows; ++r) {
            const unsigned bits = (unsigned)br.host->res[r];
            std::memcpy(&lp[r_done + r], &bits, 4);
          }
          r_done += (size_t)rows;
          st.completion_rows += rows;
        }
        for (size_t r0 = r_done; r0 < row_node.size(); r0 += kBeamCompRows) {
          const int rows = (int)std::min<size_t>(kBeamCompRows, row_node.size() - r0);
          int *slot = bp.h_stage, *tok = slot + kBeamCompRows;
          for (int r = 0; r < rows; ++r) {
            const BeamNode &x = nodes[row_node[r0 + r]];
            slot[r] = nodes[x.parent].slot;
            tok[r] = x.token;
          }
          BeamIndex si, ti;
          if (rows <= kBeamInline) {
            si = beam_inline(slot, rows); ti = beam_inline(tok, rows);
          } else {
            HIP_TRY(hipMemcpyAsync(bp.d_stage, slot, sizeof(int) * 2 * kBeamCompRows, hipMemcpyHostToDevice, s));
            si = beam_list(bp.d_stage); ti = beam_list(bp.d_stage + kBeamCompRows);
          }
          beam_enqueue_logits(m, ws, bp.e_all + (size_t)t * d.Hj, 1, bp.p, si, rows, s);
          beam_token_logp_kernel<<<(unsigned)rows, 256, 0, s>>>(ws.logits, V1, ti, (float *)bp.d_res + kBeamResComp);
          rc = check_launch("beam prefix step");
          if (rc) return rc;
          HIP_TRY(hipStreamSynchronize(s));
          std::memcpy(lp.data() + r0, (float *)bp.h_res + kBeamResComp, sizeof(float) * rows);
          st.completion_rows += rows;
        }
        std::vector<double> before(hyps.size());
        for (size_t i = 0; i < hyps.size(); ++i) before[i] = hyps[i].score;
        std::vector<char> removed(hyps.size(), 0);
        std::vector<int> chain;
        for (const Pair &pr : pairs) {
          double completion = 0.0;
          // labels in sequence order: collect the chain from B up to A, then add from A's side
          chain.clear();
          for (int x = hyps[pr.b].node; x != hyps[pr.a].node; x = nodes[x].parent) chain.push_back(x);
          for (size_t i = chain.size(); i-- > 0;) completion += (double)lp[(size_t)row_at[chain[i]].value];
          hyps[pr.b].score = beam_logaddexp(hyps[pr.b].score, before[pr.a] + completion);
          removed[pr.a] = 1;
          ++st.completions;
        }
        if (prefix_mode == WIND_PREFIX_REMOVE) {
          kept.clear();
          for (size_t i = 0; i < hyps.size(); ++i)
            if (!removed[i]) kept.push_back(hyps[i]);
          hyps.swap(kept);
        }
      }
    }

    // step 3: the K most probable (ties: shorter, then lexicographically smaller label sequence)
    {
      order.resize(hyps.size());
      for (size_t i = 0; i < hyps.size(); ++i) order[i] = (int)i;
      auto less = [&](int a, int b) {
        if (hyps[a].score != hyps[b].score) return hyps[a].score > hyps[b].score;
        const int da = nodes[hyps[a].node].depth, db = nodes[hyps[b].node].depth;
        if (da != db) return da < db;
        return tokens_of(hyps[a].node) < tokens_of(hyps[b].node);
      };
      const size_t most = std::min(order.size(), (size_t)K);
      std::partial_sort(order.begin(), order.begin() + most, order.end(), less);
      kept.clear();
      for (size_t i = 0; i < most; ++i) kept.push_back(hyps[order[i]]);
      hyps.swap(kept);
    }
    const int Bh = (int)hyps.size();

    // the survivors whose label sequence is new take a prediction-network step; then the scoring step: the window's joiner rows, P' and
    // the K best pairs of every hypothesis
    int fresh = 0, parent[kBeamMaxK], child[kBeamMaxK], tok[kBeamMaxK], slots[kBeamMaxK], fresh_of[kBeamMaxK];
    for (int b = 0; b < Bh; ++b) {
      BeamNode &nd = nodes[hyps[b].node];
      fresh_of[b] = 0;
      if (nd.slot < 0) {
        nd.slot = next_slot++;   // never used again in this search: see the resident workgroups' reads
        parent[fresh] = nodes[nd.parent].slot; child[fresh] = nd.slot; tok[fresh] = nd.token;
        fresh_of[b] = ++fresh;
      }
      slots[b] = nd.slot;
    }
    if (next_slot > bp.cap) {
      session.close();   // the pool moves
      rc = beam_pool_reserve(m, next_slot, s);
      if (rc) return rc;
    }
    if (next_slot >= 1 << kBeamSlotBits) { session.close(); session.usable = false; }
    st.decoder_steps += fresh;
    const int n = std::min(window, T - t);
    const float *scores = (const float *)bp.h_res + kBeamResScores;
    const int32_t *labels = (const int32_t *)bp.h_res + kBeamResLabels, *jumps = (const int32_t *)bp.h_res + kBeamResJumps;
    bool scored = false;
    if (session.usable) {
      unsigned words[kBeamCmdWords] = {0};
      put(words, kBeamCmdScore, fresh, Bh, n, t, K, m->opt_beam_exact ? 1 : 0);
      for (int i = 0; i < fresh; ++i) {
        words[kBeamAtParent + i] = (unsigned)parent[i]; words[kBeamAtChild + i] = (unsigned)child[i]; words[kBeamAtToken + i] = (unsigned)tok[i];
      }
      for (int b = 0; b < Bh; ++b) words[kBeamAtHyp + b] = (unsigned)(slots[b] | fresh_of[b] << kBeamSlotBits);
      rc = session.run(words, Bh * K, [&]() {
        const unsigned tag = (br.seq & 0x7FFFu) | 0x8000u;
        for (int i = 0; i < Bh * K; ++i)
          if (__atomic_load_n(&br.host->res[i], __ATOMIC_RELAXED) >> 48 != tag) return false;
        return true;
      }, &scored);
      if (rc) return rc;
      for (int i = 0; i < Bh * K && scored; ++i) {
        const unsigned long long w = br.host->res[i];
        const unsigned bits = (unsigned)w, code = (unsigned)(w >> 32) & 0x7FFFu;
        std::memcpy((float *)bp.h_res + kBeamResScores + i, &bits, 4);
        ((int32_t *)bp.h_res)[kBeamResLabels + i] = code == (unsigned)kBeamCodeNone ? -1 : (int)(code & 0x7FFu);
        ((int32_t *)bp.h_res)[kBeamResJumps + i] = code == (unsigned)kBeamCodeNone ? -1 : (int)(code >> 11);
      }
    }
    if (!scored) {
      if (fresh) beam_enqueue_decoder_step(m, fresh, parent, child, tok, s);
      beam_enqueue_logits(m, ws, bp.e_all + (size_t)t * d.Hj, n, bp.p, beam_inline(slots, Bh), Bh, s);
      beam_enqueue_topk(m, ws, n, Bh, K, (int32_t *)bp.d_res + kBeamResLabels, (int32_t *)bp.d_res + kBeamResJumps,
                        (float *)bp.d_res + kBeamResScores, s);
      rc = check_launch("beam scoring");
      if (rc) return rc;
      HIP_TRY(hipStreamSynchronize(s));
    }
    st.hyps_scored += Bh;

    if (on_round) {
      if (session.idle_callbacks >= kBeamSlowCallbacks) session.close();
      cb_len.clear(); cb_tok.clear(); cb_fr.clear(); cb_sym.clear(); cb_score.clear();
      for (const BeamHyp &h : hyps) {
        const std::vector<int> tk = tokens_of(h.node);
        cb_len.push_back((int)tk.size());
        cb_tok.insert(cb_tok.end(), tk.begin(), tk.end());
        const std::vector<int> fr = frames_of(h);
        cb_fr.insert(cb_fr.end(), fr.begin(), fr.end());
        cb_sym.push_back(h.sym);
        cb_score.push_back(h.score);
      }
      on_round(user, t, n, Bh, cb_len.data(), cb_tok.data(), cb_fr.data(), cb_score.data(), cb_sym.data(), K, labels, jumps,
               scores);
    }

    // expansion: every chosen pair becomes a hypothesis at the frame it leads to
    for (int b = 0; b < Bh; ++b) {
      for (int k = 0; k < K; ++k) {
        const int label = labels[b * K + k], jump = jumps[b * K + k];
        if (label < 0) continue;
        if (label > V || jump < 0 || jump >= n) return fail(WIND_ERR_HIP, "beam search: a pass returned a pair outside its window");
        BeamHyp nh;
        nh.score = hyps[b].score + (double)scores[b * K + k];
        if (label != V) {
          nh.node = child_node(hyps[b].node, label);
          nh.stamps = (int)stamps.size();
          stamps.push_back(BeamStamp{t + jump, hyps[b].stamps});
          nh.sym = jump == 0 ? hyps[b].sym + 1 : 1;
          int tn = t + jump;
          if (nh.sym >= S) { tn += 1; nh.sym = 0; }   // safeguard: leave the frame after S labels
          resting[tn].push_back(nh);
        } else {
          nh.node = hyps[b].node;
          nh.stamps = hyps[b].stamps;
          nh.sym = 0;
          resting[t + n].push_back(nh);
        }
      }
    }
  }

  std::vector<BeamHyp> fin = std::move(resting[T]);
  if (fin.empty()) return fail(WIND_ERR_HIP, "beam search ended without a hypothesis");
  recombine(fin);
  size_t best = 0;
  std::vector<int> best_tok = tokens_of(fin[0].node);
  for (size_t i = 1; i < fin.size(); ++i) {
    bool better = fin[i].score > fin[best].score;
    if (fin[i].score == fin[best].score) {
      const std::vector<int> tk = tokens_of(fin[i].node);
      better = tk.size() < best_tok.size() || (tk.size() == best_tok.size() && tk < best_tok);
    }
    if (better) { best = i; best_tok = tokens_of(fin[i].node); }
  }
  st.nodes = (int64_t)nodes.size();
  if (stats) *stats = st;
  *out_score = fin[best].score;
  *out_count = (int32_t)best_tok.size();
  if ((int)best_tok.size() > cap) return fail(WIND_ERR_OVERFLOW, "the best hypothesis has more labels than cap");
  const std::vector<int> best_frames = frames_of(fin[best]);
  for (size_t i = 0; i < best_tok.size(); ++i) { out_tokens[i] = best_tok[i]; out_frames[i] = best_frames[i]; }
  return WIND_OK;
}

}  // namespace

// The search keeps its hypotheses in standard containers; nothing they throw may cross the C boundary.
extern "C" int wind_beam_decode(wind_model *m, const float *enc_out, int T, int window, int K, int S, int prefix_mode,
                                int32_t *out_tokens, int32_t *out_frames, int cap, int32_t *out_count, double *out_score,
                                wind_beam_stats *stats, wind_beam_round_fn on_round, void *user, void *stream) {
  try {
    return beam_decode(m, enc_out, T, window, K, S, prefix_mode, out_tokens, out_frames, cap, out_count, out_score, stats,
                       on_round, user, stream);
  } catch (const std::exception &e) {
    return fail(WIND_ERR_HIP, std::string("beam search: ") + e.what());
  } catch (...) {
    return fail(WIND_ERR_HIP, "beam search: unknown exception");
  }
}
