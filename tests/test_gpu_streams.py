"""Calls on streams of their own, from several threads, and the asynchronous form: what one call leaves to another."""
import threading

import pytest

import wind_inputs as wi

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch

    assert torch.cuda.is_available(), "these tests need the MI355X"
    return torch


def same(a, b):
    return all(x.tolist() == y.tolist() for p, q in zip(a, b) for x, y in zip(p, q))


def load(name, B, lo, hi):
    from paper_2505_13765_amd import WindModel

    cfg = wi.scaled(wi.CONFIGS[name], B, lo, hi)
    w = wi.make_weights(cfg)
    enc, lens = wi.make_batch(cfg)
    return cfg, enc, lens, lambda: WindModel.from_config(cfg, w)


@pytest.mark.parametrize("name,B,W", [("batch32", 12, 8), ("largevocab_b128", 5, 4), ("greedy_b1", 1, 32)])
def test_first_call_on_a_stream_of_its_own(torch_cuda, name, B, W):
    """The memory that a model's first call allocates is cleared on that call's stream.  On the default stream, which has work queued
    here all the time, the clearing fell into the middle of the decode: missing labels, or workgroups that no longer found each other."""
    torch = torch_cuda
    cfg, enc, lens, make = load(name, B, 30, 60)
    d_enc, d_len = torch.from_numpy(enc).cuda(), torch.from_numpy(lens).cuda()
    m = make()
    want, resident = m.decode(d_enc, d_len, W, cfg.S), m.loop_info()[0]
    m.close()
    stop = threading.Event()

    def feed():
        a = torch.ones((2048, 2048), device="cuda")
        while not stop.is_set():
            for _ in range(20):
                a = a @ a * 1e-9
            torch.cuda.default_stream().synchronize()

    t = threading.Thread(target=feed)
    t.start()
    try:
        with torch.cuda.stream(torch.cuda.Stream()):
            for _ in range(4):
                m = make()
                for _ in range(3):
                    assert same(m.decode(d_enc, d_len, W, cfg.S), want)
                    assert m.loop_info()[0] == resident
                m.close()
    finally:
        stop.set()
        t.join()
