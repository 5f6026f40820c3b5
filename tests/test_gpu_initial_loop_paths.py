"""Edges of the initial-loop kernels: runs that share a wavefront (counts around its capacity,
a run that overflows beside one that does not), recurrences at the length of the maxima list kept
in LDS and beyond it, and segments at the size of the table of roots of unity and beyond it.

Bounds as in test_gpu_initial_loops.py: runs 1e-12, pairs exact, segments 1e-13."""
import numpy as np
import pytest

import loopgen
from oracle import ks_dns as D

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.fixture(scope="module")
def il():
    from paper_2007_06427_amd import api, initial_loops
    torch.cuda.set_device(0)
    api.init()
    return initial_loops


def rel(a, b):
    return np.max(np.abs(a - b)) / np.max(np.abs(b))


@pytest.mark.parametrize("Nx,per_wave", [(16, 32), (32, 16), (64, 8), (128, 4), (256, 2)])
def test_partly_filled_wavefronts(il, Nx, per_wave):
    rng = np.random.default_rng(Nx)
    u0 = np.stack([loopgen.random_ks_state(rng, Nx, scale=0.5) for _ in range(per_wave + 1)])
    L = 0.6 * Nx
    want = np.stack([D.integrate(u, L, 0.05, 8)[0] for u in u0])
    for n in (1, per_wave - 1, per_wave, per_wave + 1):
        u = torch.from_numpy(np.concatenate([u0[:n], np.full((1, Nx // 2 + 1), 7.0)])).to(DEV)
        il.ks_integrate(u[:n], L, 0.05, 8)
        got = u.cpu().numpy()
        assert all(rel(got[r], want[r]) < 1e-12 for r in range(n))
        assert np.all(got[n] == 7.0)  # the row after the last run


def test_an_overflowing_run_leaves_its_neighbours_alone(il):
    rng = np.random.default_rng(3)
    u0 = np.stack([loopgen.random_ks_state(rng, 64, scale=0.5) for _ in range(8)])
    clean = torch.from_numpy(u0.copy()).to(DEV)
    il.ks_integrate(clean, 39.0, 0.05, 40)
    u0[3] *= 1e200
    u = torch.from_numpy(u0).to(DEV)
    il.ks_integrate(u, 39.0, 0.05, 40)
    keep = [0, 1, 2, 4, 5, 6, 7]
    assert torch.equal(u[keep], clean[keep])
    assert not torch.isfinite(torch.view_as_real(u[3])).all()


@pytest.mark.parametrize("ns", [4096, 4098, 4100, 9000])  # 2047, 2048 and 2049 maxima, and far more
def test_recurrences_at_the_list_length(il, ns):
    rng = np.random.default_rng(ns)
    s = 1.0 + 0.01 * rng.integers(0, 50, size=ns)
    if ns < 9000:
        s[::2] -= 0.5  # every odd sample is a maximum
    norms = torch.from_numpy(s[None]).to(DEV).contiguous()
    want = D.recurrences(s, 0.1, 0.001, 1.0, 9.0)
    pairs, counts = il.ks_recurrences(norms, ns, 0.1, 0.001, 1.0, 9.0, cap=len(want) + 5)
    assert counts.item() == len(want) > 0
    assert np.array_equal(pairs.cpu().numpy()[0, :len(want)], np.array(want))
    assert np.all(pairs.cpu().numpy()[0, len(want):] == -1)


@pytest.mark.parametrize("n", [21, 4096, 4097])
def test_segments_at_the_table_size(il, n):
    rng = np.random.default_rng(n)
    snaps = rng.standard_normal((1, n + 3, 33)) + 1j * rng.standard_normal((1, n + 3, 33))
    loops, T = il.ks_segments_to_loops(torch.from_numpy(snaps).to(DEV), n + 3,
                                       torch.tensor([[0, 2, n + 2]], dtype=torch.int32, device=DEV), 0.1, 64, 10)
    want, To = D.segment_to_loop(snaps[0], 2, n + 2, 0.1, 64, 10)
    assert rel(loops.cpu().numpy()[0], want) < 1e-13 and T.item() == To
