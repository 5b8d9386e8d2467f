"""The launched kernels of wind_beam_window_scores (models and calls that the resident workgroups do not take): the choice of
a row's K largest labels, exactly, on logits that tie, and the logits' two block sizes against the fp64 oracle."""
import numpy as np
import pytest

import oracle
import wind_inputs as wi
from oracle import beam_scores as bs
from test_gpu_beam_scores import check_against_oracle, hypotheses

pytestmark = pytest.mark.gpu


def config(V, Hj=64, dtype="f32", D=64):
    return wi.WindConfig("launched", 11, 2, 70, 80, D, 64, 1, 64, Hj, V, dtype, (4,), 3, 0.5)


# 2047 / 2048: the last row of the four-wave instance and the first of the eight-wave one; 9215: the longest row; fewer labels than K; K below the number
# of waves (1 and 3 of four and eight, 7 of eight) and above
@pytest.mark.parametrize("V", [5, 63, 300, 2047, 2048, 9215])
@pytest.mark.parametrize("K", [1, 3, 7, 32])
def test_row_choice_on_ties(V, K):
    """Logits are the output bias (no weights): `top` labels share the largest value, up to all of them, more than the list of a row
    holds; the order of equal scores is earlier frame, then lower label."""
    import torch

    from paper_2505_13765_amd import WindModel

    cfg = config(V)
    w = wi.make_weights(cfg)
    w["w_out"] = np.zeros_like(w["w_out"])
    rng = np.random.default_rng(V * 100 + K)
    for top in sorted({1, min(V, 3), min(V, 40), min(V, 600), V}):
        b = (-1.0 - rng.integers(0, 3, V + 1) * 0.5).astype(np.float32)
        b[rng.choice(V, top, replace=False)] = 2.0
        b[V] = -30.0                                                     # blank: the second frame is out of reach
        w["b_out"] = b
        m = WindModel.from_config(cfg, w)
        win, g = torch.randn((2, cfg.D), device="cuda"), torch.randn((3, cfg.Hp), device="cuda")
        lab, jmp, _ = m.beam_window_scores(win, g, K)
        m.close()
        order = np.lexsort((np.arange(V), -b[:V]))[:K]
        n = len(order)
        for h in range(3):
            assert lab[h, :n].tolist() == order.tolist() and (jmp[h, :n] == 0).all(), (top, h)


# rows around the edges of 64-row blocks; 8200 labels: 257 blocks of 32 x 32 per row tile, past one per CU; 1088 units: none of those;
# 300 rows of 64 units at 1500 labels: many rows, few columns
@pytest.mark.parametrize("exact", [0, 1])
@pytest.mark.parametrize("V,Hj,n,Bh", [(8200, 64, 1, 1), (8200, 320, 16, 4), (8200, 192, 13, 5), (1500, 64, 20, 15), (1100, 1088, 7, 3), (8100, 64, 3, 2)])
def test_logit_blocks(V, Hj, n, Bh, exact):
    import torch

    from paper_2505_13765_amd import WindModel

    cfg = config(V, Hj, "bf16", 128)
    w = wi.make_weights(cfg)
    o = oracle.Oracle.from_config(cfg, w)
    m = WindModel.from_config(cfg, w)
    m.set_option("beam_exact", exact)
    enc, _ = wi.make_batch(cfg)
    g = hypotheses(o, cfg, np.random.default_rng(3), Bh, 4)
    win = np.ascontiguousarray(enc[0, 5:5 + n])
    _, _, _, full = bs.beam_window(o, win, g, 9)
    lab, jmp, sc = m.beam_window_scores(torch.from_numpy(win).cuda(), torch.from_numpy(g.astype(np.float32)).cuda(), 9)
    check_against_oracle(cfg, full, 9, lab, jmp, sc, 1e-3 if exact else 2e-2)   # split: about 16 mantissa bits of the hidden vector
    m.close()


# 60: rows that eight values do not divide; shift: inputs at an address that is no multiple of 16 bytes; 9 frames, 17 hypotheses: one
# more than a group of eight rows each; 1032, 1088: two steps of 512 values and a rest
@pytest.mark.parametrize("dtype,D,shift", [("f32", 60, 0), ("f32", 64, 1), ("bf16", 64, 0), ("bf16", 64, 3), ("f32", 1032, 0), ("bf16", 1088, 0)])
def test_projections(dtype, D, shift):
    import torch

    from paper_2505_13765_amd import WindModel

    cfg = config(1200, 64, dtype, D)
    w = wi.make_weights(cfg)
    o = oracle.Oracle.from_config(cfg, w)
    m = WindModel.from_config(cfg, w)
    enc, _ = wi.make_batch(cfg)
    g = hypotheses(o, cfg, np.random.default_rng(3), 17, 4).astype(np.float32)
    win = np.ascontiguousarray(enc[0, 5:14])

    def place(x):
        buf = torch.zeros(x.size + shift, device="cuda")
        buf[shift:] = torch.from_numpy(x).cuda().flatten()
        t = buf[shift:].view(*x.shape)
        assert t.data_ptr() % 16 == 4 * shift
        return t

    _, _, _, full = bs.beam_window(o, win, g.astype(np.float64), 9)
    lab, jmp, sc = m.beam_window_scores(place(win), place(g), 9)
    check_against_oracle(cfg, full, 9, lab, jmp, sc, 1e-4 if dtype == "f32" else 2e-2)
    m.close()
