"""Pair sums over sub-ensembles that are cut into pieces and by the chunk: every piece once,
whichever XCD it runs on.  The occupations are small whole numbers, so the sums are exact in FP32
(below 2^24) and the comparison is for equality."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


# one sub-ensemble and part of one; two, three and many, cut at the front, the end and both; pieces
# that fill the length and that do not, single pieces, sub-ensembles of one sample
@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("M", [3, 130, 300])
@pytest.mark.parametrize("E,ns,e0", [(1, 1, 0), (300, 300, 0), (512, 512, 0), (100, 1000, 450),
                                     (1000, 900, 0), (1000, 900, 450), (900, 512, 512),
                                     (2000, 300, 200), (2048, 256, 0), (2000, 256, 100), (40, 1, 3),
                                     (333, 20, 7)])
def test_every_piece_once(prec, M, E, ns, e0):
    import torch

    import paper_2503_12749_amd as mp
    rng = np.random.default_rng(M + E)
    x = rng.integers(-3, 4, (2, E, M))
    ld = mp.mp_ld_modes(M)
    dt = torch.float32 if prec == "fp32" else torch.float64
    X = torch.zeros(2, E, ld, dtype=dt, device="cuda")
    X[:, :, :M] = torch.from_numpy(x).cuda()
    n_sub = (e0 + E - 1) // ns + 2  # one more than the chunk touches
    acc = torch.full((n_sub * M * M * 2,), 0.5, dtype=torch.float64, device="cuda")
    need = mp.mp_pair_correlations_workspace(M, E, prec, ns, e0)
    ws = torch.full((max(need, 256),), 0xFF, dtype=torch.uint8, device="cuda")
    mp.mp_pair_correlations_accumulate(M, E, X, prec, n_sub, ns, e0, acc, ws)
    got = acc.cpu().numpy().view(complex).reshape(n_sub, M, M)
    z = (x[0] + 1j * x[1])
    sub = (e0 + np.arange(E)) // ns
    for s in range(n_sub):
        i = sub == s
        assert np.array_equal(got[s], z[i].T @ z[i] + (0.5 + 0.5j)), s
