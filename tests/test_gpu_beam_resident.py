"""Beam search on resident workgroups (models of one LSTM layer as wide as the joiner, up to 640 units and 1024 labels, K <= 8,
windows of at most 16 frames): the replay protocol of test_gpu_beam_search.py at the edges of the workgroups' tiles, and the
ways a search leaves them: waits that give up, workgroups that have gone idle, another call that takes its turn."""
import threading
import time

import numpy as np
import pytest

import oracle
import wind_inputs as wi
from test_gpu_beam_search import replay, torch_cuda  # noqa: F401

pytestmark = pytest.mark.gpu


def small(H, V, T, K, S):
    cfg = wi.WindConfig("beam_resident", 40 + H, 1, T, T, 64, 64, 1, H, H, V, "bf16", (8,), S, 0.7)
    return cfg, wi.sharpened(wi.make_weights(cfg, blank_bias=2.0, pred_gain=4.0), 4.0)


# one column past a tile of 16, all tiles and the one past them, a single tile; one to 16 frames; one to eight hypotheses; every width
@pytest.mark.parametrize("H,V,T,N,K,S,exact", [(128, 16, 20, 16, 8, 4, 1), (128, 1024, 18, 7, 5, 3, 1), (256, 31, 24, 1, 3, 2, 1), (384, 1023, 18, 16, 4, 3, 1),
                                               (512, 1008, 17, 9, 8, 3, 0), (640, 1024, 16, 16, 8, 3, 1), (640, 1024, 21, 5, 1, 3, 1), (640, 300, 18, 13, 6, 4, 0)])
def test_replay_at_the_edges(torch_cuda, H, V, T, N, K, S, exact):  # noqa: F811
    from paper_2505_13765_amd import WindModel

    cfg, w = small(H, V, T, K, S)
    o = oracle.Oracle.from_config(cfg, w)
    m = WindModel.from_config(cfg, w)
    m.set_option("beam_exact", exact)
    enc, _ = wi.make_batch(cfg)
    stats = replay(o, m, torch_cuda, np.ascontiguousarray(enc[0]), N, K, S, "keep", (2e-4 if exact else 4e-2) * 4, free_run=False)
    print(f"H={H} V={V} N={N} K={K} exact={exact}: {stats}")
    route = m.route_counts()
    assert route.beam_commands > 0 and route.beam_gave_up == 0   # the passes of the search that was replayed were the workgroups'
    m.close()


def test_the_ways_out(torch_cuda):  # noqa: F811
    """Launches only; a wait that gives up at once (the whole search then runs on launches); workgroups that go idle between two
    passes: the same choices every time, scores to rounding."""
    from paper_2505_13765_amd import WindModel

    cfg, w = small(256, 100, 40, 4, 3)
    m = WindModel.from_config(cfg, w)
    m.set_option("beam_exact", 1)
    e = torch_cuda.from_numpy(wi.make_batch(cfg)[0][0]).cuda()
    here = m.beam_decode(e, 8, 4, 3)
    m.set_option("loop_kernel", 0)
    launches = m.beam_decode(e, 8, 4, 3)
    m.set_option("loop_kernel", 1)
    limit = 1 << 21
    m.set_option("loop_spin_limit", 0)
    given_up = m.beam_decode(e, 8, 4, 3)
    m.set_option("loop_spin_limit", limit)

    class Slow(list):
        def append(self, x):
            time.sleep(0.004 if len(self) % 5 == 0 else 0.0)
            super().append(x)

    idle = m.beam_decode(e, 8, 4, 3, trace=Slow())
    again = m.beam_decode(e, 8, 4, 3)
    route = m.route_counts()
    assert route.beam_gave_up == 1 and route.beam_idle > 0 and route.beam_launches >= 4
    assert route.beam_commands >= here[3].rounds + idle[3].rounds + again[3].rounds
    for other in (launches, given_up, idle, again):
        assert other[0].tolist() == here[0].tolist() and other[1].tolist() == here[1].tolist()
        assert abs(other[2] - here[2]) < 1e-3 * max(1.0, abs(here[2]))
    assert again[2] == here[2] and idle[2] == here[2] and given_up[2] == launches[2]
    m.close()


def test_other_calls_take_their_turn(torch_cuda):  # noqa: F811
    """A greedy decode in resident groups on another thread and stream goes in between the search's passes, and both get their results."""
    from paper_2505_13765_amd import WindModel

    cfg, w = small(640, 1024, 120, 4, 3)
    searcher, decoder = WindModel.from_config(cfg, w), WindModel.from_config(cfg, w)
    enc = torch_cuda.from_numpy(wi.make_batch(cfg)[0]).cuda()
    lens = torch_cuda.tensor([120], dtype=torch_cuda.int32, device="cuda")
    want_b = searcher.beam_decode(enc[0], 16, 4, 3)
    want_g = decoder.decode(enc, lens, 8, 3)
    stop, wrong, calls = threading.Event(), [], [0]

    def greedy():
        with torch_cuda.cuda.stream(torch_cuda.cuda.Stream()):
            while not stop.is_set():
                got = decoder.decode(enc, lens, 8, 3)
                calls[0] += 1
                if got[0][0].tolist() != want_g[0][0].tolist():
                    wrong.append(calls[0])

    th = threading.Thread(target=greedy)
    th.start()
    try:
        for _ in range(4):
            got = searcher.beam_decode(enc[0], 16, 4, 3)
            assert got[0].tolist() == want_b[0].tolist() and got[2] == want_b[2]
    finally:
        stop.set()
        th.join()
    assert not wrong and calls[0] > 4
    route = searcher.route_counts()
    assert route.beam_gave_up == 0 and route.beam_launches > 5   # they left for the decodes, and came back
    searcher.close()
    decoder.close()


# hypotheses that leave groups empty, fill one each, and fill all; windows of one to 16 frames; columns at the tiles' edges
@pytest.mark.parametrize("H,V,n,Bh,K,exact", [(128, 16, 16, 1, 8, 1), (128, 1024, 5, 9, 4, 1), (256, 31, 1, 8, 1, 0), (384, 992, 16, 64, 8, 1),
                                              (512, 1023, 11, 17, 5, 0), (640, 1024, 16, 16, 8, 1), (640, 1024, 16, 61, 8, 0)])
def test_one_scoring_step(torch_cuda, H, V, n, Bh, K, exact):  # noqa: F811
    """Against the oracle, and the same choices and scores (to rounding) as the launches that take every other shape; buffers that are
    aligned to four bytes only take those.  Workgroups that cannot meet: the same sums in launches that need not, to the bit, as the
    static entry point has them."""
    from oracle import beam_scores as bs
    from paper_2505_13765_amd import WindModel
    from test_gpu_beam_scores import check_against_oracle, hypotheses

    torch = torch_cuda
    cfg, w = small(H, V, 16, K, 4)
    o = oracle.Oracle.from_config(cfg, w)
    m = WindModel.from_config(cfg, w)
    m.set_option("beam_exact", exact)
    enc = wi.make_batch(cfg)[0][0, :n]
    dec = hypotheses(o, cfg, np.random.default_rng(H + V), Bh, 4).astype(np.float32)
    _, _, _, full = bs.beam_window(o, enc, dec.astype(np.float64), K)
    e, d = torch.from_numpy(np.ascontiguousarray(enc)).cuda(), torch.from_numpy(dec).cuda()
    tol = (2e-4 if exact else 4e-2) * 4
    got = m.beam_window_scores(e, d, K)
    check_against_oracle(cfg, full, K, *got, tol)
    odd = torch.empty(d.numel() + 1, device="cuda")[1:].view(d.shape).copy_(d)
    unaligned = m.beam_window_scores(e, odd, K)
    m.set_option("loop_spin_limit", 0)
    given_up = m.beam_window_scores(e, d, K)
    m.set_option("loop_spin_limit", 1 << 21)
    again = m.beam_window_scores(e, d, K)
    route = m.route_counts()
    assert route.scores_resident == 2 and route.scores_gave_up == 1
    static = [torch.full((Bh, K), -9, dtype=t, device="cuda") for t in (torch.int32, torch.int32, torch.float32)]
    m.beam_window_scores_static(e, d, K, static)
    torch.cuda.synchronize()
    # Other orders of the fp32 sums; without `exact` a hidden unit may also round to the other bf16 value: 2^-8 of a weight of the
    # output layer (4 / sqrt(H)) times a unit of about one, 6e-4 at 640 units, a few at most
    assert np.allclose(unaligned[2], got[2], atol=2e-4 if exact else 4e-3, rtol=1e-5)
    assert (unaligned[0] != got[0]).mean() <= 0.02   # near-ties
    for other in (again, given_up, [t.cpu().numpy() for t in static]):
        for a, b in zip(got, other):
            assert a.tobytes() == b.tobytes()
    m.close()


@pytest.mark.parametrize("exact", [0, 1])
@pytest.mark.parametrize("H,V", [(256, 100), (640, 1024)])
def test_a_scoring_step_of_values_that_are_not_finite(torch_cuda, H, V, exact):  # noqa: F811
    """Infinities and NaN in a frame or in a hypothesis: the pairs, and the places of scores that are not numbers, of the launches that take every
    other shape."""
    from paper_2505_13765_amd import WindModel

    torch = torch_cuda
    cfg, w = small(H, V, 16, 4, 4)
    m = WindModel.from_config(cfg, w)
    m.set_option("beam_exact", exact)
    for what, value in (("frame", np.inf), ("frame", -np.inf), ("frame", np.nan), ("hypothesis", np.inf), ("hypothesis", -np.inf), ("hypothesis", np.nan),
                        ("every frame", np.inf), ("every hypothesis", np.inf)):
        g = torch.Generator(device="cpu").manual_seed(3)
        e, d = torch.randn((8, cfg.D), generator=g), torch.tanh(torch.randn((10, H), generator=g))
        if what.startswith("every"):
            (e if "frame" in what else d)[:] = value
        elif what == "frame":
            e[3, 5] = value
        else:
            d[4, 7] = value
        e, d = e.cuda(), d.cuda()
        runs = []
        for resident in (1, 0):
            m.set_option("loop_kernel", resident)
            runs.append(m.beam_window_scores(e, d, 4))
        here, there = runs
        assert np.array_equal(here[0], there[0]) and np.array_equal(here[1], there[1]), (what, value)
        assert np.array_equal(np.isfinite(here[2]), np.isfinite(there[2])), (what, value)
        ok = np.isfinite(there[2])
        assert np.allclose(here[2][ok], there[2][ok], atol=2e-4 if exact else 4e-3, rtol=1e-5), (what, value)   # see test_one_scoring_step
    assert m.route_counts().scores_resident == 8 and m.route_counts().scores_gave_up == 0
    m.close()


def test_steps_and_searches_after_a_failed_meeting(torch_cuda):  # noqa: F811
    """Workgroups that could not meet are not asked again at once: each failure costs the wait for them."""
    from paper_2505_13765_amd import WindModel

    torch = torch_cuda
    cfg, w = small(256, 100, 16, 4, 3)
    m = WindModel.from_config(cfg, w)
    e, d = torch.from_numpy(wi.make_batch(cfg)[0][0]).cuda(), torch.tanh(torch.randn((10, 256), device="cuda"))
    want = m.beam_window_scores(e, d, 4)
    search = m.beam_decode(e, 8, 4, 3)
    m.set_option("loop_spin_limit", 0)
    for k in range(300):   # one failure, 256 steps without, another
        got = m.beam_window_scores(e, d, 4)
        assert all(a.tobytes() == b.tobytes() for a, b in zip(want, got))
    for k in range(10):    # and 8 searches
        again = m.beam_decode(e, 8, 4, 3)
        assert again[0].tolist() == search[0].tolist() and again[1].tolist() == search[1].tolist()
    route = m.route_counts()
    assert (route.scores_resident, route.scores_gave_up, route.beam_gave_up) == (1, 2, 2)
    m.set_option("loop_spin_limit", 1 << 21)
    m.beam_window_scores(e, d, 4)
    assert m.route_counts().scores_resident == 2
    m.close()


def test_callbacks_that_wait_for_the_gpu(torch_cuda):  # noqa: F811
    """A callback that synchronises with the device waits for the workgroups too, until they leave: the first few times, and no longer than a pass
    with launches takes."""
    from paper_2505_13765_amd import WindModel

    torch = torch_cuda
    cfg, w = small(640, 1024, 60, 4, 3)
    m = WindModel.from_config(cfg, w)
    e = torch.from_numpy(wi.make_batch(cfg)[0][0]).cuda()
    want = m.beam_decode(e, 16, 4, 3)
    waits = []

    class Waiting(list):
        def append(self, x):
            t = time.perf_counter()
            torch.cuda.synchronize()
            waits.append(time.perf_counter() - t)
            super().append(x)

    before = m.route_counts()
    got = m.beam_decode(e, 16, 4, 3, trace=Waiting())
    after = m.route_counts()
    assert got[0].tolist() == want[0].tolist() and got[2] == want[2] and len(waits) == got[3].rounds > 40
    print(f"{len(waits)} callbacks, wait {1e6 * np.median(waits):.0f} us, {after.beam_idle - before.beam_idle} idle")
    assert after.beam_idle - before.beam_idle <= 4 and after.beam_gave_up == 0
    assert np.median(waits) < 200e-6   # 1 ms of an idle launch each before; a synchronisation alone takes 10 us
    m.close()
