"""Runs of more maxima than the list in LDS holds, around the number of samples whose maxima fit
in its bits (131072) and around whole words of them: pairs and counts equal the definition's, also
where the caller's room runs out."""
import numpy as np
import pytest

from oracle import ks_dns as D

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("ns", [6335, 6336, 6337, 131071, 131072, 131073])
def test_pairs_equal_the_definition(ns):
    from paper_2007_06427_amd import api, initial_loops as il
    torch.cuda.set_device(0)
    api.init()
    s = 1.0 + 0.01 * np.random.default_rng(ns).integers(0, 50, size=(2, ns))
    norms = torch.from_numpy(s).to(DEV)
    for cap in (200000, 50):
        pairs, counts = il.ks_recurrences(norms, ns, 0.1, 0.003, 0.5, 2.0, cap=cap)
        for r in range(2):
            want = D.recurrences(s[r], 0.1, 0.003, 0.5, 2.0)
            assert counts[r].item() == len(want) > 50
            got = pairs[r].cpu().numpy()
            assert np.array_equal(got[:len(want)], np.array(want)[:cap])
            assert np.all(got[len(want):] == -1)
