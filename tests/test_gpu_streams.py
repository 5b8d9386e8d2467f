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


def async_buffers(torch, m, B, T, W, S):
    out = [torch.zeros(s, dtype=torch.int32, device="cuda") for s in ((B, T * S), (B, T * S), (B,))]
    ws = torch.full((m.workspace_bytes(B, T, W) + 256,), 0xFF, dtype=torch.uint8, device="cuda")
    return out, ws[(-ws.data_ptr()) % 256:][: m.workspace_bytes(B, T, W)]


def taken(out):
    tok, frm, cnt = (x.cpu().numpy() for x in out)
    return [tok[b, :n] for b, n in enumerate(cnt)], [frm[b, :n] for b, n in enumerate(cnt)]


@pytest.mark.parametrize("name,dtype,B", [("batch32", "bf16", 5), ("batch32", "f32", 2), ("tiny", "f32", 3)])
def test_asynchronous_decode_needs_no_meeting(torch_cuda, name, dtype, B):
    """An asynchronous call of a batch must not depend on its workgroups being on the chip together (here: they give up at
    once, set from the host): nobody would decode it again."""
    torch = torch_cuda
    from paper_2505_13765_amd import WindModel

    cfg = wi.scaled(wi.CONFIGS[name], B, 30, 60).replace(dtype=dtype)
    m = WindModel.from_config(cfg, wi.make_weights(cfg))
    enc, lens = wi.make_batch(cfg)
    d_enc, d_len = torch.from_numpy(enc).cuda(), torch.from_numpy(lens).cuda()
    m.set_option("loop_kernel", 0)
    want = m.decode(d_enc, d_len, 8, cfg.S)
    m.set_option("loop_kernel", 1)
    m.set_option("loop_spin_limit", 0)
    T = enc.shape[1]
    out, ws = async_buffers(torch, m, B, T, 8, cfg.S)
    m.greedy_decode_async(d_enc, d_len, 8, cfg.S, *out, ws, T * (cfg.S + 1) + 2)
    m.stats()
    assert same(taken(out), want)
    m.close()


@pytest.mark.parametrize("name,B,W", [("greedy_b1", 1, 16), ("greedy_b1", 1, 32), ("batch32", 4, 8), ("tiny", 2, 4)])
def test_captured_asynchronous_decode(torch_cuda, name, B, W):
    """A captured asynchronous decode, launched several times with synchronous calls of the same model on another batch in between: every
    launch gives the eager result, and the synchronous calls theirs."""
    torch = torch_cuda
    cfg, enc, lens, make = load(name, B, 20, 40)
    m = make()
    d_enc, d_len = torch.from_numpy(enc).cuda(), torch.from_numpy(lens).cuda()
    e2 = d_enc.flip(1).contiguous()
    l2 = torch.full_like(d_len, enc.shape[1])
    want, want2 = m.decode(d_enc, d_len, W, cfg.S), m.decode(e2, l2, W, cfg.S)
    m.decode(d_enc, d_len, W, cfg.S)
    iterations = int(m.stats().iterations)
    out, ws = async_buffers(torch, m, B, enc.shape[1], W, cfg.S)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        m.greedy_decode_async(d_enc, d_len, W, cfg.S, *out, ws, iterations)
    g.replay()
    torch.cuda.synchronize()
    assert m.stats().iterations == iterations
    for _ in range(3):
        for x in out:
            x.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert same(taken(out), want)
        assert same(m.decode(e2, l2, W, cfg.S), want2)
    m.close()
