"""What is timed when the decoder's speed is followed over changes: whole calls through the public entry points of
`paper_2505_13765_amd.WindModel`, over the range of sizes the library is used at.

The models are the workloads of `wind_inputs` (random-init weights, blank rate calibrated), the encoder outputs are
N(0, 1) frames of ragged batches padded to the longest length that the program takes.  As in a serving program a model is loaded
once and then decodes one batch after another, each in buffers of its own; so the models are kept here, and a
state is one batch: its frames, its lengths and the buffers its labels go to.
"""
from __future__ import annotations

import numpy as np
import torch

import wind_inputs as wi
from paper_2505_13765_amd import WindModel

# kind "decode": wind_greedy_decode with window W, or wind_sequential_decode (W = 0) | "scores": one scoring step of the beam
# search for B hypotheses on a window of W frames | "beam": a whole beam search over one utterance of `hi` frames.
# model: a configuration of wind_inputs, its weights kept in bf16 or in fp32.  lo, hi: range of the utterances' lengths.


def listed():
    return [
        # the smallest model, fp32: one short utterance (the quick check a user runs first)
        {"name": "tiny_f32", "kind": "decode", "model": "tiny", "dtype": "f32", "B": 1, "lo": 64, "hi": 64, "W": 4},
        # one utterance of ten seconds: a voice command, or a chunk of a stream
        {"name": "short_b1", "kind": "decode", "model": "greedy_b1", "dtype": "bf16", "B": 1, "lo": 125, "hi": 125, "W": 8},
        # one long utterance, the benchmark's headline, and the same frame by frame (the standard algorithm)
        {"name": "greedy_b1", "kind": "decode", "model": "greedy_b1", "dtype": "bf16", "B": 1, "lo": 1000, "hi": 1000, "W": 16},
        {"name": "sequential_b1", "kind": "decode", "model": "greedy_b1", "dtype": "bf16", "B": 1, "lo": 1000, "hi": 1000, "W": 0},
        # small batches, as of an interactive service: a few long utterances; an odd number of short ones and an odd window
        {"name": "batch4", "kind": "decode", "model": "batch32", "dtype": "bf16", "B": 4, "lo": 200, "hi": 1500, "W": 8},
        {"name": "batch13_ragged", "kind": "decode", "model": "batch32", "dtype": "bf16", "B": 13, "lo": 37, "hi": 611, "W": 5},
        # the batched workloads: a medium batch, a large vocabulary with two LSTM layers, many labels per frame
        {"name": "batch32", "kind": "decode", "model": "batch32", "dtype": "bf16", "B": 32, "lo": 200, "hi": 1500, "W": 8},
        {"name": "largevocab_b128", "kind": "decode", "model": "largevocab_b128", "dtype": "bf16", "B": 128, "lo": 500, "hi": 2000, "W": 16},
        {"name": "lowblank_b256", "kind": "decode", "model": "lowblank_b256", "dtype": "bf16", "B": 256, "lo": 100, "hi": 1000, "W": 16},
        # fp32 weights on a model of ordinary size (a reference run, or a model that must not be rounded)
        {"name": "f32_batch8", "kind": "decode", "model": "batch32", "dtype": "f32", "B": 8, "lo": 100, "hi": 600, "W": 8},
        # beam search: its scoring step as a caller with a search of its own uses it, and the whole search
        {"name": "beam_scores", "kind": "scores", "model": "greedy_b1", "dtype": "bf16", "B": 16, "lo": 16, "hi": 16, "W": 16, "K": 8},
        {"name": "beam_search", "kind": "beam", "model": "greedy_b1", "dtype": "bf16", "B": 1, "lo": 250, "hi": 250, "W": 16, "K": 4},
    ]


def _log_int(rng, lo, hi):
    """An integer of [lo, hi], even over its logarithm."""
    return max(lo, min(hi, int(round(lo * (hi / lo) ** rng.random()))))


def draw(rng):
    what = rng.choice(("tiny", "one", "one", "few", "few", "few", "largevocab", "lowblank", "f32", "scores", "beam"))
    if what == "scores":
        return {"kind": "scores", "model": rng.choice(("greedy_b1", "largevocab_b128")), "dtype": "bf16", "B": rng.randint(1, 32), "lo": 1, "hi": 1,
                "W": rng.randint(1, 16), "K": rng.randint(1, 16)}
    if what == "beam":
        T = _log_int(rng, 30, 250)
        return {"kind": "beam", "model": "greedy_b1", "dtype": "bf16", "B": 1, "lo": T, "hi": T, "W": rng.randint(4, 16), "K": rng.randint(2, 8)}
    if what == "tiny":
        T = _log_int(rng, 16, 200)
        return {"kind": "decode", "model": "tiny", "dtype": "f32", "B": rng.randint(1, 3), "lo": max(1, T // 2), "hi": T, "W": rng.randint(1, 8)}
    if what == "one":
        T = _log_int(rng, 40, 1500)
        return {"kind": "decode", "model": "greedy_b1", "dtype": "bf16", "B": rng.choice((1, 1, 1, 2)), "lo": max(1, 3 * T // 4), "hi": T,
                "W": rng.choice((0, 2, 3, 4, 8, 8, 11, 16))}
    if what == "few":
        hi = _log_int(rng, 80, 1500)
        return {"kind": "decode", "model": "batch32", "dtype": "bf16", "B": _log_int(rng, 3, 64), "lo": max(1, hi // rng.randint(2, 9)), "hi": hi,
                "W": rng.choice((0, 2, 4, 5, 8, 8, 16))}
    if what == "f32":
        hi = _log_int(rng, 60, 600)
        return {"kind": "decode", "model": "batch32", "dtype": "f32", "B": rng.randint(1, 8), "lo": max(1, hi // rng.randint(2, 6)), "hi": hi,
                "W": rng.choice((2, 4, 8))}
    name, hi_most, b_most = ("largevocab_b128", 2000, 128) if what == "largevocab" else ("lowblank_b256", 1000, 256)
    hi = _log_int(rng, 200, hi_most)
    return {"kind": "decode", "model": name, "dtype": "bf16", "B": _log_int(rng, 8, b_most), "lo": max(1, hi // rng.randint(2, 8)), "hi": hi,
            "W": rng.choice((4, 8, 16, 16))}


_models = {}


def _config(case):
    return wi.CONFIGS[case["model"]].replace(dtype=case["dtype"])


def _model(case):
    """The model of a case, loaded once.  Beam search takes the headline model with its output layer times eight, whose soft-max
    is peaked like a trained model's."""
    key = (case["model"], case["dtype"], case["kind"] == "beam")
    if key not in _models:
        cfg = _config(case)
        w = wi.make_weights(cfg)
        _models[key] = WindModel.from_config(cfg, wi.sharpened(w, 8.0) if case["kind"] == "beam" else w)
    return _models[key]


def prepare(case, seed):
    cfg, model = _config(case), _model(case)
    gen = torch.Generator(device="cuda").manual_seed(int(seed) * 1000003 + 17)

    def frames(*shape):
        x = torch.randn(shape, generator=gen, dtype=torch.float32, device="cuda")
        return x.bfloat16().float() if cfg.dtype == "bf16" else x   # an encoder in bf16 hands over bf16 values

    state = {"kind": case["kind"], "model": model, "W": case["W"] or None, "S": cfg.S, "K": case.get("K", 0)}
    if case["kind"] == "scores":
        state["enc"] = frames(case["W"], cfg.D)
        state["dec"] = torch.tanh(torch.randn((case["B"], cfg.Hp), generator=gen, dtype=torch.float32, device="cuda"))
        pairs = torch.zeros((2, case["B"], case["K"]), dtype=torch.int32, device="cuda")
        state["pairs"], state["scores"] = pairs, torch.zeros((case["B"], case["K"]), dtype=torch.float32, device="cuda")
        return state
    rng = np.random.default_rng([int(seed), case["B"], case["lo"], case["hi"]])
    lengths = rng.integers(case["lo"], case["hi"] + 1, size=case["B"]).astype(np.int32)
    T = case["hi"]
    if case["kind"] == "beam":
        state["enc"] = frames(T, cfg.D)
        return state
    state["enc"] = frames(case["B"], T, cfg.D)
    state["lengths"] = torch.from_numpy(lengths).cuda()
    # one allocation for what the call returns: labels, their frames, their number
    B, cap = case["B"], T * cfg.S
    state["out"] = out = torch.zeros(2 * B * cap + B, dtype=torch.int32, device="cuda")
    state["tokens"], state["frames"] = out[: B * cap].view(B, cap), out[B * cap: 2 * B * cap].view(B, cap)
    state["counts"] = out[2 * B * cap:]
    return state


def run(state):
    m = state["model"]
    if state["kind"] == "decode":
        m.greedy_decode(state["enc"], state["lengths"], state["W"], state["S"], state["tokens"], state["frames"], state["counts"])
        return state["out"]
    if state["kind"] == "scores":
        m.beam_window_scores(state["enc"], state["dec"], state["K"], (state["pairs"][0], state["pairs"][1], state["scores"]))
        return state["pairs"], state["scores"]
    tokens, frames, score, _ = m.beam_decode(state["enc"], state["W"], state["K"], state["S"])
    labels = np.full((2, state["enc"].shape[0] * state["S"]), -1, np.int32)
    labels[0, : len(tokens)], labels[1, : len(frames)] = tokens, frames
    return labels, float(score)


def work(case):
    """Per frame: its projection; per joiner evaluation of the frame-by-frame algorithm (every frame ends in a blank or in S
    labels, so about frames / blank rate of them): the output layer; per label: one prediction-network step and its projection.
    Bytes: the frames and the weights read once, the labels written once."""
    cfg = _config(case)
    size = 2 if cfg.dtype == "bf16" else 4
    layers = [((cfg.E if l == 0 else cfg.Hp) + cfg.Hp) * 4 * cfg.Hp for l in range(cfg.L)]
    out_layer, pred = (cfg.V + 1) * cfg.Hj, cfg.Hp * cfg.Hj
    if case["kind"] == "scores":
        n, B = case["W"], case["B"]
        return {"flops": 2.0 * (n * cfg.D * cfg.Hj + B * pred + n * B * out_layer),
                "bytes": 4.0 * (n * cfg.D + B * cfg.Hp + 3 * B * case["K"]) + size * (cfg.D * cfg.Hj + pred + out_layer)}
    frames = case["B"] * (case["lo"] + case["hi"]) / 2.0
    evals = frames / cfg.blank_rate
    labels = evals - frames
    if case["kind"] == "beam":   # every expanded label sequence takes a step, every frame is scored for each of the K survivors
        evals, labels = frames * case["K"], frames * case["K"] * (1 - cfg.blank_rate)
    return {"flops": 2.0 * (frames * cfg.D * cfg.Hj + evals * out_layer + labels * (sum(layers) + pred)),
            "bytes": 4.0 * frames * cfg.D + size * (cfg.D * cfg.Hj + sum(layers) + pred + out_layer) + 8.0 * labels}


def tolerance(case):
    """Labels and frames are decided on fp32 sums: where two logits are closer than those sums' rounding either label is right, and the
    rest of that utterance then differs.  Scores are logarithms of probabilities from logits with bf16 operands."""
    if case["kind"] == "decode":
        return {"rel": 0.0, "differ": 0.002}
    return {"rel": 1e-3, "max": 1e-2, "differ": 0.01}
