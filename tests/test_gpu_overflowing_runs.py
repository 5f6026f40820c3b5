"""A run that overflows ends non-finite in every retained mode, the mean's real and imaginary part
among them, as the integration of the definitions does, and keeps zeros beyond the band."""
import numpy as np
import pytest

import loopgen
from oracle import ks_dns as D

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("Nx", [16, 32, 64, 128, 256])
def test_every_mode_of_an_overflowed_run_is_non_finite(Nx):
    from paper_2007_06427_amd import api, initial_loops as il
    torch.cuda.set_device(0)
    api.init()
    rng = np.random.default_rng(Nx)
    u0 = 1e200 * loopgen.random_ks_state(rng, Nx, scale=0.5)
    u0[0] += 0.25 + 0.5j
    K = (Nx - 1) // 3
    with np.errstate(all="ignore"):
        want = D.integrate(u0, 0.6 * Nx, 0.05, 2)[0]
    u = torch.from_numpy(u0[None]).to(DEV)
    norms = torch.zeros(1, 2, dtype=torch.float64, device=DEV)
    snaps = torch.zeros(1, 2, Nx // 2 + 1, dtype=torch.complex128, device=DEV)
    il.ks_integrate(u, 0.6 * Nx, 0.05, 2, 1, False, norms, snaps)
    assert snaps[0, 0, 0].item() == u0[0]  # the first sample is the state as given
    for got in (u[0].cpu().numpy(), snaps[0, 1].cpu().numpy()):
        for part in (got.real, got.imag):
            assert not np.isfinite(part[:K + 1]).any()
            assert np.all(part[K + 1:] == 0.0)
    assert not np.isfinite(want.real[:K + 1]).any() and not np.isfinite(want.imag[:K + 1]).any()
