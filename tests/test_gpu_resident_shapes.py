"""The resident form at every shape it takes (block sizes of 64 to 512 threads, pairs with and
without a second row, exchange space shared with the intermediates): its steps and its gradient
equal the per-pass kernels' bit for bit, and a gradient can be recorded into a HIP graph
as the first call of its shape."""
import numpy as np
import pytest

import loopgen

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

DEV = "cuda:0"
SHAPES = [(M, N) for M in (8, 16, 32, 64, 128) for N in (8, 16, 32, 64, 128, 256, 512)]


@pytest.fixture(scope="module")
def api():
    from paper_2007_06427_amd import api as A
    torch.cuda.set_device(0)
    A.init()
    prev = A.set_resident(A.RESIDENT_ALWAYS)
    yield A
    A.set_resident(prev)


def state(Nx, Ns, n):
    rng = np.random.default_rng(Nx * 1000 + Ns)
    u = np.stack([loopgen.random_band_field(rng, Nx, Ns, scale=0.3) for _ in range(n)])
    u[:, :, 0] += 0.1j * rng.standard_normal((n, Ns))  # read through its Hermitian part
    return torch.from_numpy(u).to(DEV), torch.from_numpy(rng.uniform(20.0, 80.0, n)).to(DEV)


@pytest.mark.parametrize("Nx,Ns", SHAPES, ids=[f"{a}x{b}" for a, b in SHAPES])
def test_steps_and_gradient_equal_per_pass(api, Nx, Ns):
    if not api.resident_supported(Nx, Ns):
        assert api.step_form(Nx, Ns, 1) == "per-pass"
        return
    L, dtau = 0.5 * Nx, 1e-6
    u, T = state(Nx, Ns, 3)
    b = api.Batch([(L, Nx, Ns)] * 3)
    for scheme in (0, 1):
        ua, Ta, Ja = u.clone(), T.clone(), torch.zeros(3, 3, dtype=torch.float64, device=DEV)
        api.loop_step(ua, Ta, L, dtau if scheme else 1e-12, scheme, 3, J_hist=Ja)
        pool, Tb, Jb = u.reshape(-1).clone(), T.clone(), torch.zeros(3, 3, dtype=torch.float64, device=DEV)
        b.step(pool, Tb, dtau if scheme else 1e-12, scheme, 3, J_hist=Jb)
        assert torch.equal(Ja, Jb) and torch.equal(Ta, Tb) and torch.equal(ua.reshape(-1), pool)
    for n in (1, 3):
        res = api.loop_adjoint_grad(u[:n], T[:n], L)
        api.set_resident(api.RESIDENT_NEVER)
        ref = api.loop_adjoint_grad(u[:n], T[:n], L)
        api.set_resident(api.RESIDENT_ALWAYS)
        assert all(torch.equal(x, y) for x, y in zip(res, ref))


def test_first_gradient_under_capture(api):
    """No earlier call of this shape: the kernel's LDS limit is raised while recording."""
    u, T = state(64, 128, 1)
    ws = api.Workspace(api.workspace_bytes(64, 128, 1))
    out = torch.empty_like(u), torch.empty(1, dtype=torch.float64, device=DEV), torch.empty(1, dtype=torch.float64, device=DEV)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        for o, x in zip(out, api.loop_adjoint_grad(u, T, 30.0, ws=ws)):
            o.copy_(x)
    for k in range(3):
        u.mul_(1.0 + 0.1 * k)
        g.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(o, x) for o, x in zip(out, api.loop_adjoint_grad(u, T, 30.0)))
