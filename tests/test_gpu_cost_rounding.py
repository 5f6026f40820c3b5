"""The rounding of the cost J where it comes from the transforms alone: loops of an amplitude whose
products outweigh the linear part, against long double. Twiddle powers formed by products have a
magnitude that is off by their rounding, which the inverse and the forward transform do not cancel:
with one stage of them per transform J is off by 2.5e-16 to 3e-16 (rms) at 16 and 32 points and
by 6e-16 at 128 points, with two by 4.3e-16 to 4.9e-16 and 6.5e-16 to 6.9e-16. The bounds lie between."""
import numpy as np
import pytest

import loopgen

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

LD = np.longdouble


def cost(u, T, L, Nx, Ns):
    """J in long double, with the wave numbers as double precision has them."""
    Kx, Ks = (Nx - 1) // 3, (Ns - 1) // 3
    j, k = np.arange(Nx // 2 + 1), np.fft.fftfreq(Ns, 1.0 / Ns)
    mask = (np.abs(k) <= Ks)[:, None] & (j <= Kx)[None, :]
    u = u.astype(np.clongdouble) * mask
    u[:, 0] = (u[:, 0] + np.roll(u[::-1, 0], 1).conj()) / 2
    q, om = (2.0 * np.pi * j / L).astype(LD)[None, :], (2.0 * np.pi * k).astype(LD)[:, None]

    def phys(v):
        return np.fft.irfft2(v, s=(Ns, Nx), norm="forward")

    r = (-(1j * om / LD(T)) * u - np.fft.rfft2(phys(u) * phys(1j * q * u), norm="forward") + (q**2 - q**4) * u) * mask
    return LD(L) / 2 * (np.where(j == 0, 1, 2)[None, :] * np.abs(r) ** 2).sum()


@pytest.mark.skipif(np.finfo(LD).nmant < 60, reason="long double is no wider than double here")
@pytest.mark.parametrize("Nx,Ns,bound", [(16, 16, 3.6e-16), (16, 32, 3.6e-16), (32, 16, 3.6e-16), (32, 32, 3.6e-16),
                                         (128, 64, 6.3e-16), (256, 32, 6.3e-16)])
def test_cost_of_products(Nx, Ns, bound):
    from paper_2007_06427_amd import api
    torch.cuda.set_device(0)
    api.init()
    rng, n, L = np.random.default_rng(Nx + Ns), 64, 0.5 * Nx
    u = np.stack([loopgen.random_band_field(rng, Nx, Ns, scale=1e6) for _ in range(n)])
    T = rng.uniform(20.0, 80.0, n)
    ref = [cost(u[i], T[i], L, Nx, Ns) for i in range(n)]
    ud, Td = torch.from_numpy(u).to("cuda:0"), torch.from_numpy(T).to("cuda:0")
    for J in (api.loop_cost(ud, Td, L), api.loop_adjoint_grad(ud, Td, L)[2]):
        e = [float((LD(J[i].item()) - ref[i]) / ref[i]) for i in range(n)]
        assert np.sqrt(np.mean(np.square(e))) < bound
