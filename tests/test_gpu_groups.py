"""The resident groups (one per XCD) that decode small batches of one-layer models, against the oracle and, counter for
counter, against the graph of per-step kernels: one to four slots per group, slots that take a second utterance,
empty utterances, windows that fill a row tile and that do not, vocabularies with empty and ragged column parts, and every width the
kernel is built for."""
import numpy as np
import pytest

import oracle
import wind_inputs as wi
from parity import compare_batch

pytestmark = pytest.mark.gpu


# H, V, B, W: groups of one, two, three, four slots; 41 and 70 utterances: slots take a second and a third; the row
# tiles of a group's workgroups (1, 2, 4) come from slots x window; 2 utterances of 640: groups of 20 workgroups
@pytest.mark.parametrize("H,V,B,W", [(640, 1024, 1, 16), (640, 1024, 2, 7), (640, 1024, 3, 1), (640, 1000, 9, 16), (640, 1024, 17, 11), (640, 1024, 41, 16),
                                     (512, 77, 70, 5), (384, 300, 33, 8), (256, 1, 12, 9), (128, 1024, 26, 13), (128, 31, 8, 16)])
def test_resident_groups(H, V, B, W):
    import torch
    from paper_2505_13765_amd import WindModel

    assert torch.cuda.is_available(), "this test needs the MI355X"
    cfg = wi.WindConfig("groups", 40 + B, B, 1, 75, 64, 64, 1, H, H, V, "bf16", (W,), 3, 0.7)
    w = wi.make_weights(cfg, blank_bias=2.0 if V > 1 else 0.0, pred_gain=4.0)
    enc, lens = wi.make_batch(cfg)
    lens[0], lens[B // 2] = 0 if B > 2 else 33, 1 if B > 4 else lens[B // 2]
    for b in range(B):
        enc[b, lens[b]:] = np.nan
    m = WindModel.from_config(cfg, w)
    d_enc, d_len = torch.from_numpy(enc).cuda(), torch.from_numpy(lens).cuda()
    res = []
    for loop in (1, 0):
        m.set_option("loop_kernel", loop)
        toks, frs = m.decode(d_enc, d_len, W, cfg.S)
        assert m.loop_info()[0] == (0 if not loop else 40 if B == 2 and H == 640 else 32 * min(B, 8))
        st = m.stats()
        res.append((toks, frs, (st.iterations, st.windows, st.rows, st.useful_rows, st.labels, st.forced_advances, list(st.jump_hist))))
    print(f"groups H={H} V={V} B={B} W={W}: {res[0][2][:6]}", flush=True)
    excluded = compare_batch(oracle.Oracle.from_config(cfg, w), enc, lens, cfg.S, res[0][0], res[0][1])
    assert excluded <= 1 + B // 16
    assert res[0][2][4] == sum(len(t) for t in res[0][0]) > 0
    if excluded == 0:   # a near-tie may fall either way on either route
        assert all(a.tolist() == b.tolist() for k in (0, 1) for a, b in zip(res[0][k], res[1][k]))
        assert res[0][2] == res[1][2]
    m.close()


def test_two_streams_and_threads_take_turns():
    """Resident kernels of several models, called from several threads on streams of their own, must not wait for each other's CUs."""
    import threading

    import torch
    from paper_2505_13765_amd import WindModel

    cfg = wi.scaled(wi.CONFIGS["batch32"], 12, 30, 80)
    w = wi.make_weights(cfg)
    enc, lens = wi.make_batch(cfg)
    d_enc, d_len = torch.from_numpy(enc).cuda(), torch.from_numpy(lens).cuda()
    models = [WindModel.from_config(cfg, w) for _ in range(3)]
    ref = models[0].decode(d_enc, d_len, 8, cfg.S)
    torch.cuda.synchronize()
    bad = []

    def work(m):
        with torch.cuda.stream(torch.cuda.Stream()):
            for _ in range(4):
                toks, frs = m.decode(d_enc, d_len, 8, cfg.S)
                if not all(a.tolist() == b.tolist() for r, g in zip(ref, (toks, frs)) for a, b in zip(r, g)):
                    bad.append(m)

    threads = [threading.Thread(target=work, args=(m,)) for m in models]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad
    for m in models:
        m.close()
