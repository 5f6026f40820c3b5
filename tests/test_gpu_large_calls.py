"""Calls of more than 128 MiB of work space write intermediates over those they have read: every
entry point's results for a set of loops of that size equal, bit for bit, those of calls on a few
of the loops, which keep them apart."""
import numpy as np
import pytest

import loopgen

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

DEV = "cuda:0"
FEW = 2


@pytest.fixture(scope="module")
def api():
    from paper_2007_06427_amd import api as A
    torch.cuda.set_device(0)
    A.init()
    return A


def loops(api, Nx, Ns, nl):
    assert api.workspace_bytes(Nx, Ns, nl) > 128 << 20 > api.workspace_bytes(Nx, Ns, FEW)
    rng = np.random.default_rng(Nx + Ns)
    few = [torch.from_numpy(loopgen.random_band_field(rng, Nx, Ns, scale=0.3)) for _ in range(FEW)]
    u = torch.stack([few[i % FEW] for i in range(nl)]).to(DEV)
    return u.contiguous(), torch.linspace(30.0, 60.0, nl, dtype=torch.float64, device=DEV)


def calls(api, u, T, L, grid):
    """Every entry point's outputs for the loops u, with the loop as the first axis."""
    nl = len(T)
    out = {"cost": (api.loop_cost(u, T, L),), "residual": (api.loop_residual(u, T, L),),
           "adjoint": api.loop_adjoint_grad(u, T, L), "cost_grad": api.loop_cost_grad(u, T, L),
           "expanded": api.loop_expanded_grad(u, T, L)}
    for name in ("loop_step", "loop_step_expanded", "loop_step_xi"):
        v, t, J = u.clone(), T.clone(), torch.zeros(3, nl, dtype=torch.float64, device=DEV)
        getattr(api, name)(v, t, L, 1e-6, api.IMEX, 3, J_hist=J)
        out[name] = v, t, J.t()
    band = api.to_band(u)
    for layout, x in ((api.LAYOUT_RFFT, u), (api.LAYOUT_BAND, band)):
        g = grid if layout == api.LAYOUT_BAND else None
        for us in (None, api.saved_u(nl, *grid, DEV)):
            J, dJdT, r = api.loop_cost_fwd(x, T, L, layout, g, usave=us)
            out["bwd", layout, us is None] = J, dJdT, r, *api.loop_cost_bwd(x, T, L, r, dJdT, None, layout, g, usave=us)
    return out


@pytest.mark.parametrize("Nx,Ns,nl", [(256, 1024, 25), (512, 256, 60), (64, 64, 4000), (16, 256, 3000)])
def test_equals_small_calls(api, Nx, Ns, nl):
    u, T = loops(api, Nx, Ns, nl)
    prev = api.set_resident(api.RESIDENT_NEVER)
    try:
        big = calls(api, u, T, 0.5 * Nx, (Nx, Ns))
        for at in (0, nl // 2, nl - FEW):
            part = slice(at, at + FEW)
            few = calls(api, u[part].contiguous(), T[part].contiguous(), 0.5 * Nx, (Nx, Ns))
            for k in few:
                assert len(big[k]) == len(few[k])
                assert all(torch.equal(x[part], y) for x, y in zip(big[k], few[k])), (k, at)
    finally:
        api.set_resident(prev)


@pytest.mark.parametrize("streams", [0, 2, 3, 4])
def test_batch_equals_small_batches(api, streams):
    shapes = [(256, 1024)] * 20 + [(512, 256)] * 12 + [(64, 256)] * 20 + [(64, 64)] * 8
    rng = np.random.default_rng(5)
    fields = {s: torch.from_numpy(loopgen.random_band_field(rng, *s, scale=0.3)) for s in set(shapes)}

    def step(shapes, T):
        b = api.Batch([(0.5 * Nx, Nx, Ns) for Nx, Ns in shapes])
        if streams:
            b.set_schedule(b.STREAMS, streams)
        pool, t = b.pack([fields[s] for s in shapes]), T.clone()
        J = torch.zeros(3, len(shapes), dtype=torch.float64, device=DEV)
        b.step(pool, t, 1e-6, api.IMEX, 3, J_hist=J)
        return b, pool, t, J

    T = torch.linspace(30.0, 60.0, len(shapes), dtype=torch.float64, device=DEV)
    b, pool, t, J = step(shapes, T)
    assert b.ws.numel() > 128 << 20
    views = b.unpack(pool)
    for at in (0, 19, 20, 32, 52):
        part = slice(at, at + 2)
        c, p, tc, Jc = step(shapes[part], T[part])
        assert torch.equal(t[part], tc) and torch.equal(J[:, part], Jc), at
        assert all(torch.equal(x, y) for x, y in zip(views[part], c.unpack(p))), at
