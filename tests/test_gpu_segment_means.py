"""Segments cut with the fewest time modes (kc = 0, the mean alone, which takes a path of its own,
and kc = 1) with a table of roots and beyond it, against the definition to 1e-13."""
import numpy as np
import pytest

from oracle import ks_dns as D

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("Nx,Ns", [(8, 8), (64, 64), (1024, 8)])
@pytest.mark.parametrize("kc", [0, 1])
@pytest.mark.parametrize("n", [1, 3, 9, 300, 4096, 4097])
def test_lowest_time_modes(n, kc, Nx, Ns):
    from paper_2007_06427_amd import api, initial_loops as il
    torch.cuda.set_device(0)
    api.init()
    H = Nx // 2 + 1
    rng = np.random.default_rng(n + kc)
    snaps = rng.standard_normal((2, n + 3, H)) + 1j * rng.standard_normal((2, n + 3, H))
    triples = torch.tensor([[0, 2, n + 2], [1, 0, n], [1, 3, n + 3]], dtype=torch.int32, device=DEV)
    loops, T = il.ks_segments_to_loops(torch.from_numpy(snaps).to(DEV), n + 3, triples, 0.1, Ns, kc)
    for l, (r, a, b) in enumerate(triples.tolist()):
        got = loops[l].cpu().numpy()
        if n <= 2 * kc:  # too short for its modes: refused
            assert T[l].item() == 0.0 and np.all(got == 0.0)
            continue
        want, To = D.segment_to_loop(snaps[r], a, b, 0.1, Ns, kc)
        assert np.max(np.abs(got - want)) < 1e-13 * np.max(np.abs(want)) and T[l].item() == To
