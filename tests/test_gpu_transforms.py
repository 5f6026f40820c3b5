"""Every transform length of the row and column passes, in each form that uses them: three loops
(an odd number, so that the last block of a pass is partly empty) of n x 32 and 32 x n for
n = 8 .. 1024, fields filling the whole band, against the FP64 oracle.

Bound: a transform of n points errs by at most a few log2(n) units in the last place of its
norm, and a gradient passes through four of them and products of full-band fields; the per-step
bound of the method, 1e-12 normwise, holds at every length."""
import numpy as np
import pytest

import loopgen
from oracle import ks_loop as K

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TOL = 1e-12
DEV = "cuda:0"
LENGTHS = [8, 16, 32, 64, 128, 256, 512, 1024]
SHAPES = [(n, 32) for n in LENGTHS] + [(32, n) for n in LENGTHS if n != 32]


@pytest.fixture(scope="module")
def api():
    from paper_2007_06427_amd import api as A
    torch.cuda.set_device(0)
    A.init()
    return A


def wrel(a, b):
    w = np.full(a.shape[-1], 2.0)
    w[0] = 1.0
    return np.sqrt(np.sum(w * np.abs(a - b) ** 2)) / np.sqrt(np.sum(w * np.abs(b) ** 2))


def loops(Nx, Ns, odd):
    rng = np.random.default_rng(Nx + 3 * Ns)
    draw = loopgen.random_xi_symmetric_field if odd else loopgen.random_band_field
    return np.stack([draw(rng, Nx, Ns, scale=0.3) for _ in range(3)]), np.array([17.0, 40.0, 95.0]), 0.4 * Nx


@pytest.mark.parametrize("Nx,Ns", SHAPES, ids=[f"{a}x{b}" for a, b in SHAPES])
def test_every_length_matches_oracle(api, Nx, Ns):
    u, T, L = loops(Nx, Ns, False)
    ud, Td = torch.from_numpy(u).to(DEV), torch.from_numpy(T).to(DEV)
    G, dT, J = (x.cpu().numpy() for x in api.loop_adjoint_grad(ud, Td, L))
    ref = [K.adjoint_grad(u[i], T[i], L) for i in range(3)]
    for i in range(3):
        assert wrel(G[i], ref[i][0]) < TOL
        assert abs(J[i] - ref[i][2]) <= TOL * ref[i][2]
    api.loop_step(ud, Td, L, 1e-9, api.IMEX, 2)
    for i in range(3):
        uo, To, _ = K.step(u[i], T[i], L, 1e-9, K.IMEX, 2)
        assert wrel(ud.cpu().numpy()[i], uo) < TOL


@pytest.mark.parametrize("Nx,Ns", [s for s in SHAPES if s[0] <= 512], ids=[f"{a}x{b}" for a, b in SHAPES if a <= 512])
def test_every_length_centre_symmetric_and_expanded(api, Nx, Ns):
    u, T, L = loops(Nx, Ns, True)
    ud, Td = torch.from_numpy(u).to(DEV), torch.from_numpy(T).to(DEV)
    api.loop_step_xi(ud, Td, L, 1e-9, api.IMEX, 2)
    for i in range(3):
        uo, To, _ = K.step(u[i], T[i], L, 1e-9, K.IMEX, 2)
        assert wrel(ud.cpu().numpy()[i], uo) < TOL
        assert abs(Td[i].item() - To) <= TOL * To
    if (Nx - 1) // 3 * (2 * ((Ns - 1) // 3) + 1) < Ns:
        return  # the expanded form's row sums do not fit these few columns
    u, T, L = loops(Nx, Ns, False)
    G, dT, J = (x.cpu().numpy() for x in api.loop_expanded_grad(torch.from_numpy(u).to(DEV), torch.from_numpy(T).to(DEV), L))
    for i in range(3):
        Go, dTo, Jo = K.expanded_grad(u[i], T[i], L)
        assert wrel(G[i], Go) < TOL
        assert abs(J[i] - Jo) <= TOL * Jo
