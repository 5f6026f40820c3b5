"""A plan that is being recorded into a HIP graph can be stepped on another stream at the same
time, with a work space of its own: the step completes, the recording stays whole, and both give
the plain steps' bits; each replay is compared, with eager steps between them."""
import ctypes

import numpy as np
import pytest

import loopgen

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

DEV = "cuda:0"
SHAPES = [(32, 32), (64, 64), (64, 128), (32, 128), (32, 512), (64, 256)]


@pytest.fixture(scope="module")
def api():
    from paper_2007_06427_amd import api as A
    torch.cuda.set_device(0)
    A.init()
    return A


@pytest.mark.parametrize("streams", [0, 3])
def test_eager_step_during_a_capture(api, streams):
    from paper_2007_06427_amd import _lib
    rng = np.random.default_rng(streams)
    b = api.Batch([(0.5 * Nx, Nx, Ns) for Nx, Ns in SHAPES])
    if streams:
        b.set_schedule(b.STREAMS, streams)
    u = b.pack([torch.from_numpy(loopgen.random_band_field(rng, Nx, Ns, scale=0.3)) for Nx, Ns in SHAPES])
    T = torch.from_numpy(rng.uniform(20.0, 80.0, b.nloops)).to(DEV)
    side = torch.cuda.Stream()
    hs, P = ctypes.c_void_p(side.cuda_stream), ctypes.c_void_p
    ws = torch.empty(b.ws.numel(), dtype=torch.uint8, device=DEV)
    ue, Te, ug, Tg, us, Ts = u.clone(), T.clone(), u.clone(), T.clone(), u.clone(), T.clone()
    torch.cuda.synchronize()
    api.check(_lib.lib().loop_batch_workspace_init(b._plan, P(ws.data_ptr()), ws.numel(), hs), "init")

    def step_aside():
        api.check(_lib.lib().loop_batch_step(b._plan, P(Ts.data_ptr()), P(us.data_ptr()), 1e-6, api.IMEX, 2, None,
                                             P(ws.data_ptr()), ws.numel(), hs), "step")

    prev = api.set_resident(api.RESIDENT_ALWAYS)
    try:
        b.step(ue, Te, 1e-6, api.IMEX, 2)  # the plain step, and the kernels' set-up
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            b.step(ug, Tg, 1e-6, api.IMEX, 2)
            step_aside()
        side.synchronize()
        assert torch.equal(us, ue) and torch.equal(Ts, Te)
        for i in range(3):
            g.replay()
            torch.cuda.synchronize()
            assert torch.equal(ug, ue) and torch.equal(Tg, Te)
            step_aside()  # on the plan's streams again
            side.synchronize()
            b.step(ue, Te, 1e-6, api.IMEX, 2)
            torch.cuda.synchronize()
            assert torch.equal(us, ue) and torch.equal(Ts, Te)
    finally:
        api.set_resident(prev)
    assert b.status() == 0
