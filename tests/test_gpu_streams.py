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


def backlog(torch, stream):
    """Some 0.4 s of matrix products on the stream, and an event behind them."""
    a = torch.ones((8192, 8192), device="cuda")
    with torch.cuda.stream(stream):
        for _ in range(40):
            a = a @ a * 1e-9
        behind = torch.cuda.Event()
        behind.record()
    return behind


def test_no_host_thread_waits_for_anothers_stream(torch_cuda):
    """Resident kernels take turns on the GPU.  While a synchronous call waits behind the work that its stream has queued, an asynchronous
    call of another model on another stream returns at once, and a small fp32 model, whose workgroups wait for nobody, decodes."""
    import time

    torch = torch_cuda
    cfg, enc, lens, make = load("greedy_b1", 1, 60, 60)
    tiny_cfg, tiny_enc, tiny_lens, make_tiny = load("tiny", 2, 30, 60)
    m, other, tiny = make(), make(), make_tiny()
    d_enc, d_len, t_enc, t_len = (torch.from_numpy(x).cuda() for x in (enc, lens, tiny_enc, tiny_lens))
    want, want_tiny = m.decode(d_enc, d_len, 16, cfg.S), tiny.decode(t_enc, t_len, 4, tiny_cfg.S)
    assert same(other.decode(d_enc, d_len, 16, cfg.S), want)
    out, ws = async_buffers(torch, other, 1, enc.shape[1], 16, cfg.S)
    torch.cuda.synchronize()
    beside = 0
    for _ in range(6):   # streams may share a hardware queue, and the tiny decode then comes behind the products after all
        s1, s2, s3, got = torch.cuda.Stream(), torch.cuda.Stream(), torch.cuda.Stream(), []
        behind = backlog(torch, s1)

        def work():
            with torch.cuda.stream(s1):
                got.append(m.decode(d_enc, d_len, 16, cfg.S))

        t = threading.Thread(target=work)
        t.start()
        time.sleep(0.02)   # it has put its kernels on its stream
        with torch.cuda.stream(s2):
            other.greedy_decode_async(d_enc, d_len, 16, cfg.S, *out, ws, enc.shape[1] * (cfg.S + 1) + 2)
        assert not behind.query()
        with torch.cuda.stream(s3):
            assert same(tiny.decode(t_enc, t_len, 4, tiny_cfg.S), want_tiny)
        beside += not behind.query()
        t.join()
        assert other.stats().labels == sum(map(len, want[0]))
        assert same(got[0], want) and same(taken(out), want)
        assert m.loop_info()[0] == other.loop_info()[0] == 32
        if beside:
            break
    assert beside
    for x in (m, other, tiny):
        x.close()


def test_groups_do_not_wait_long_for_their_places(torch_cuda):
    """While a kernel that outlasts the call (here: a captured asynchronous decode of one utterance, whose launches the caller keeps
    apart or not) holds some CUs of every XCD, a batch is decoded by the per-step kernels, not after it."""
    import time

    torch = torch_cuda
    from paper_2505_13765_amd import WindModel

    one = wi.scaled(wi.CONFIGS["greedy_b1"], 1, 5000, 5000)
    m = WindModel.from_config(one, wi.make_weights(one, blank_bias=-50.0))   # labels on every frame: 1.3 s
    d_one, l_one = torch.randn((1, 5000, one.D), device="cuda"), torch.full((1,), 5000, dtype=torch.int32, device="cuda")
    out, ws = async_buffers(torch, m, 1, 5000, 32, one.S)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        m.greedy_decode_async(d_one, l_one, 32, one.S, *out, ws, 5000 * (one.S + 1) + 2)
    cfg, enc, lens, make = load("batch32", 12, 30, 60)
    batch = make()
    d_enc, d_len = torch.from_numpy(enc).cuda(), torch.from_numpy(lens).cuda()
    batch.set_option("loop_kernel", 0)
    want = batch.decode(d_enc, d_len, 8, cfg.S)
    batch.set_option("loop_kernel", 1)
    assert same(batch.decode(d_enc, d_len, 8, cfg.S), want) and batch.loop_info()[0] == 256
    pair_cfg, p_enc, p_len, make_pair = load("greedy_b1", 2, 30, 60)
    pair = make_pair()
    p_enc, p_len = torch.from_numpy(p_enc).cuda(), torch.from_numpy(p_len).cuda()
    want_pair = pair.decode(p_enc, p_len, 16, pair_cfg.S)
    assert pair.loop_info()[0] == 64
    beside = False
    for _ in range(6):   # streams may share a hardware queue, and the batch then comes behind the other kernel
        s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
        with torch.cuda.stream(s1):
            g.replay()
            behind = torch.cuda.Event()
            behind.record()
        time.sleep(0.02)
        assert not behind.query()
        with torch.cuda.stream(s2):
            start = time.perf_counter()
            assert same(batch.decode(d_enc, d_len, 8, cfg.S), want)
            took = time.perf_counter() - start
            # two utterances: the loop kernel, which meets at grid barriers, finds places for its 40 workgroups
            assert same(pair.decode(p_enc, p_len, 16, pair_cfg.S), want_pair)
        beside = not behind.query()
        torch.cuda.synchronize()
        assert m.stats().labels == 5000 * one.S == int(out[2][0])   # the other kernel was not disturbed
        if beside:
            break
    assert beside and pair.loop_info()[0] == 40
    assert took < 0.1 and batch.loop_info()[0] == 0   # 14 ms; the limit of the later waits is 0.4 s
    assert same(batch.decode(d_enc, d_len, 8, cfg.S), want) and batch.loop_info()[0] == 256
    for x in (m, batch, pair):
        x.close()


def test_a_call_waits_on_the_gpu_for_an_asynchronous_one(torch_cuda):
    """An asynchronous call leaves its turn behind on its stream: a batch of another model on another stream, called while the first
    is still queued, finds its places afterwards.  Both run as resident groups."""
    torch = torch_cuda
    cfg, enc, lens, make = load("greedy_b1", 2, 40, 60)
    m = make()
    bcfg, benc, blens, make_batch = load("batch32", 12, 30, 60)
    batch = make_batch()
    d_enc, d_len, b_enc, b_len = (torch.from_numpy(x).cuda() for x in (enc, lens, benc, blens))
    want, want_batch = m.decode(d_enc, d_len, 8, cfg.S), batch.decode(b_enc, b_len, 8, bcfg.S)
    out, ws = async_buffers(torch, m, 2, enc.shape[1], 8, cfg.S)
    torch.cuda.synchronize()
    for _ in range(3):
        s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
        behind = backlog(torch, s1)
        with torch.cuda.stream(s1):
            m.greedy_decode_async(d_enc, d_len, 8, cfg.S, *out, ws, enc.shape[1] * (cfg.S + 1) + 2)
        assert not behind.query()
        with torch.cuda.stream(s2):
            assert same(batch.decode(b_enc, b_len, 8, bcfg.S), want_batch)
        assert behind.query()   # it came behind the asynchronous call
        m.stats()
        assert same(taken(out), want)
        assert (m.loop_info()[0], batch.loop_info()[0]) == (64, 256)
    m.close()
    batch.close()
