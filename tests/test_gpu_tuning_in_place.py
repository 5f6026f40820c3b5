"""The tuner on a plan large enough that its steps write their intermediates in place (above
128 MiB of work space), with and without loops of the resident form beside: the state is left as
it was, nothing turns non-finite, and the tuned plan steps as variant 0 on the per-pass kernels."""
import numpy as np
import pytest

import loopgen

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("small", [0, 40])
def test_tuned_plan_steps_the_same_bits(small):
    from paper_2007_06427_amd import api
    torch.cuda.set_device(0)
    api.init()
    rng = np.random.default_rng(small)
    shapes = [(128, 512)] * 140 + [(64, 128)] * small
    b = api.Batch([(0.5 * Nx, Nx, Ns) for Nx, Ns in shapes])
    assert b.ws.numel() > 128 << 20
    spec = {s: torch.from_numpy(loopgen.random_band_field(rng, *s, scale=0.3)) for s in set(shapes)}
    pool = b.pack([spec[s] for s in shapes])
    T = torch.from_numpy(rng.uniform(20.0, 80.0, b.nloops)).to(DEV)
    p0, T0 = pool.clone(), T.clone()
    rep = b.autotune(pool, T, reps=8)
    assert torch.equal(pool, p0) and torch.equal(T, T0) and b.status() == 0
    assert all(t > 0 for times in rep["pass_us"].values() for t in times.values())
    b.step(pool, T, 1e-6, api.IMEX, 3)
    ref = api.Batch(b.shapes)
    ref.set_schedule(ref.PER_PASS)
    prev = api.set_resident(api.RESIDENT_NEVER)
    try:
        for p in range(5):
            ref.set_variant(p, 0)
        ref.step(p0, T0, 1e-6, api.IMEX, 3)
    finally:
        api.set_resident(prev)
    assert torch.equal(pool, p0) and torch.equal(T, T0)
    assert b.status() == 0 and ref.status() == 0
