"""Batches whose small loops take the resident form inside loop_batch_step: only small loops
(every block size), only large ones, and both, on the per-pass and the streams schedules, equal
the steps with the resident form off bit for bit, with the form taken always and where it pays
(calls on both sides of each line of that rule); recorded into a HIP graph, replayed between
eager work, too; and two threads stepping one plan with work spaces of their own."""
import threading

import numpy as np
import pytest

import loopgen

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

DEV = "cuda:0"
SMALL = [(8, 8), (16, 8), (32, 32), (16, 64), (64, 64), (32, 128), (64, 128), (128, 64), (8, 512), (32, 64)]
LARGE = [(64, 256), (128, 128), (32, 512), (256, 16)]
MIXES = {"small": SMALL, "one-class": [(32, 32)] * 3, "large": LARGE, "both": SMALL + LARGE, "one-each": [(64, 64), (64, 256)]}


@pytest.fixture(scope="module")
def api():
    from paper_2007_06427_amd import api as A
    torch.cuda.set_device(0)
    A.init()
    return A


def batch(api, shapes):
    rng = np.random.default_rng(len(shapes))
    b = api.Batch([(0.5 * Nx, Nx, Ns) for Nx, Ns in shapes])
    pool = b.pack([torch.from_numpy(loopgen.random_band_field(rng, Nx, Ns, scale=0.3)) for Nx, Ns in shapes])
    return b, pool, torch.from_numpy(rng.uniform(20.0, 80.0, len(shapes))).to(DEV)


def step(api, b, pool, T, nsteps=3):
    pool, T = pool.clone(), T.clone()
    J = torch.zeros(nsteps, b.nloops, dtype=torch.float64, device=DEV)
    b.step(pool, T, 1e-6, api.IMEX, nsteps, J_hist=J)
    return pool, T, J


@pytest.mark.parametrize("mix", list(MIXES))
def test_equals_the_per_pass_kernels(api, mix):
    b, pool, T = batch(api, MIXES[mix])
    prev = api.set_resident(api.RESIDENT_NEVER)
    try:
        ref = step(api, b, pool, T)
    finally:
        api.set_resident(prev)
    for schedule, k in ((b.PER_PASS, None), (b.STREAMS, 2), (b.STREAMS, 3), (b.STREAMS, 4)):
        b.set_schedule(schedule, k)
        for mode in (api.RESIDENT_ALWAYS, api.RESIDENT_AUTO, api.RESIDENT_ALWAYS):
            prev = api.set_resident(mode)
            try:
                out = step(api, b, pool, T)
            finally:
                api.set_resident(prev)
            assert all(torch.equal(x, y) for x, y in zip(out, ref)), (mix, schedule, k, mode)
    assert b.status() == 0


@pytest.mark.parametrize("streams", [0, 2, 3, 4])
@pytest.mark.parametrize("mix,nsteps", [("small", 1), ("small", 2), ("small", 3), ("small", 4), ("many", 2), ("many", 4),
                                        ("many", 10)])
def test_where_it_pays(api, mix, nsteps, streams):
    """Short and long calls, few loops and enough of them (47 MB per step) to be taken out."""
    b, pool, T = batch(api, {"many": [(64, 128)] * 60 + [(32, 128)] * 60 + [(64, 256)]}.get(mix, MIXES.get(mix)))
    if streams:
        b.set_schedule(b.STREAMS, streams)
    got = step(api, b, pool, T, nsteps)
    prev = api.set_resident(api.RESIDENT_NEVER)
    try:
        ref = step(api, b, pool, T, nsteps)
    finally:
        api.set_resident(prev)
    assert all(torch.equal(x, y) for x, y in zip(got, ref))


@pytest.fixture
def always(api):
    prev = api.set_resident(api.RESIDENT_ALWAYS)
    yield
    api.set_resident(prev)


@pytest.mark.parametrize("mix", ["small", "both"])
def test_graph_replays(api, always, mix):
    b, pool, T = batch(api, MIXES[mix])
    b.set_schedule(b.STREAMS, 2)
    pg, Tg = pool.clone(), T.clone()
    step(api, b, pool, T)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        b.step(pg, Tg, 1e-6, api.IMEX, 2)
    pe, Te = pool.clone(), T.clone()
    for _ in range(3):
        g.replay()
        torch.cuda.synchronize()
        b.step(pe, Te, 1e-6, api.IMEX, 2)
        assert torch.equal(pg, pe) and torch.equal(Tg, Te)


def test_two_threads_step_one_plan(api, always):
    """The per-pass schedule, a work space and a stream for each thread."""
    import ctypes

    from paper_2007_06427_amd import _lib
    b, pool, T = batch(api, MIXES["both"])
    ref = step(api, b, pool, T, 8)
    out, fail = {}, []

    def work(i):
        try:
            s = torch.cuda.Stream()
            with torch.cuda.stream(s):
                ws = torch.empty(b.ws.numel(), dtype=torch.uint8, device=DEV)
                p, t = pool.clone(), T.clone()
                hs, P = ctypes.c_void_p(s.cuda_stream), ctypes.c_void_p
                api.check(_lib.lib().loop_batch_workspace_init(b._plan, P(ws.data_ptr()), ws.numel(), hs), "init")
                for _ in range(4):
                    api.check(_lib.lib().loop_batch_step(b._plan, P(t.data_ptr()), P(p.data_ptr()), 1e-6, api.IMEX, 2,
                                                         None, P(ws.data_ptr()), ws.numel(), hs), "step")
                s.synchronize()
                out[i] = p, t
        except Exception as e:  # reported by the main thread
            fail.append(e)

    torch.cuda.synchronize()
    threads = [threading.Thread(target=work, args=(i,)) for i in range(2)]
    [t.start() for t in threads]
    [t.join() for t in threads]
    assert not fail, fail
    # four calls of two steps: each call makes column 0 canonical, so they agree with one call
    # of eight steps to rounding and with each other bit for bit
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
    assert torch.allclose(out[0][1], ref[1], rtol=1e-13, atol=0)
