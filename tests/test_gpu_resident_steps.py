"""Steps of the resident form against the per-pass kernels, bit for bit, at every shape that has the
form, with both schemes: the batch that gives the reference runs with the form off, and the
kernel trace shows that each side took its own kernels."""
import numpy as np
import pytest

import loopgen

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

DEV = "cuda:0"
SHAPES = [(M, N) for M in (8, 16, 32, 64, 128) for N in (8, 16, 32, 64, 128, 256, 512)]
NSTEPS = 3


@pytest.fixture(scope="module")
def api():
    from paper_2007_06427_amd import api as A
    torch.cuda.set_device(0)
    A.init()
    return A


def run(api, mode, step):
    """step()'s tensors under a resident mode, and the names of the kernels it launched."""
    prev = api.set_resident(mode)
    try:
        with api.trace() as tr:
            out = step()
            torch.cuda.synchronize()
    finally:
        api.set_resident(prev)
    return out, {k.split("<")[0] for k in tr.kernels}


def test_shapes_of_the_form(api):
    assert sum(api.resident_supported(*s) for s in SHAPES) == 29


@pytest.mark.parametrize("scheme", [0, 1])
@pytest.mark.parametrize("Nx,Ns", SHAPES, ids=[f"{a}x{b}" for a, b in SHAPES])
def test_steps_equal_per_pass(api, Nx, Ns, scheme):
    if not api.resident_supported(Nx, Ns):
        assert api.step_form(Nx, Ns, 1) == "per-pass"
        return
    rng = np.random.default_rng(Nx * 1000 + Ns + scheme)
    n, L, dtau = 3, 0.5 * Nx, 1e-6  # dtau |lambda| up to 0.1: both schemes are stable
    u0 = np.stack([loopgen.random_band_field(rng, Nx, Ns, scale=0.3) for _ in range(n)])
    u0[:, :, 0] += 0.1j * rng.standard_normal((n, Ns))  # read through its Hermitian part
    u0, T0 = torch.from_numpy(u0).to(DEV), torch.from_numpy(rng.uniform(20.0, 80.0, n)).to(DEV)
    b = api.Batch([(L, Nx, Ns)] * n)

    def uniform(k):
        def step():
            u, T, J = u0[:k].clone(), T0[:k].clone(), torch.zeros(NSTEPS, k, dtype=torch.float64, device=DEV)
            api.loop_step(u, T, L, dtau, scheme, NSTEPS, J_hist=J)
            return u, T, J
        return step

    def batch():
        u, T, J = u0.clone(), T0.clone(), torch.zeros(NSTEPS, n, dtype=torch.float64, device=DEV)
        b.step(u.view(-1), T, dtau, scheme, NSTEPS, J_hist=J)
        return u, T, J

    ref, names = run(api, api.RESIDENT_NEVER, batch)
    assert "k_rag" in names and not any("resident" in k for k in names)
    assert not torch.equal(ref[0], u0) and all(torch.isfinite(x.abs()).all() for x in ref)
    got, names = run(api, api.RESIDENT_ALWAYS, batch)
    assert names == {"k_resident_batch"}
    assert all(torch.equal(x, y) for x, y in zip(got, ref))
    for k in (1, n):
        got, names = run(api, api.RESIDENT_ALWAYS, uniform(k))
        assert names == {"k_resident"}
        assert torch.equal(got[0], ref[0][:k]) and torch.equal(got[1], ref[1][:k]) and torch.equal(got[2], ref[2][:, :k])
    one, names = run(api, api.RESIDENT_NEVER, uniform(1))
    assert "k_rowB" in names and not any("resident" in k for k in names)
    assert torch.equal(one[0], ref[0][:1]) and torch.equal(one[1], ref[1][:1]) and torch.equal(one[2], ref[2][:, :1])
