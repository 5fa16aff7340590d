"""An infinite occupation in the last sample of a sub-ensemble whose length is no multiple of the
32-sample slab gives the sums that it gives in a whole slab: the padding of the slab takes no
part."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("part", [0, 1])
def test_padding_of_a_slab_takes_no_part(prec, part):
    import torch

    import paper_2503_12749_amd as mp
    M, j = 200, 190
    dt = torch.float32 if prec == "fp32" else torch.float64
    ld, sums = mp.mp_ld_modes(M), []
    for E, at in ((37, 36), (37, 10), (64, 36)):  # last of the padded slab, inside, whole slabs
        X = torch.zeros(2, E, ld, dtype=dt, device="cuda")
        X[:, :37, :M] = 1.0
        X[part, at, j] = float("inf")
        acc = torch.zeros(M * M * 2, dtype=torch.float64, device="cuda")
        nb = mp.mp_pair_correlations_workspace(M, E, prec, E, 0)
        ws = torch.empty(max(nb, 256), dtype=torch.uint8, device="cuda")
        mp.mp_pair_correlations_accumulate(M, E, X, prec, 1, E, 0, acc, ws)
        sums.append(acc.cpu().numpy().reshape(M, M, 2))
    assert np.array_equal(sums[0], sums[1], equal_nan=True)
    # one part infinite: the real part of its products is infinite, not NaN
    assert np.all(np.isinf(np.delete(sums[0][:, j, 0], j)))
    finite = np.delete(np.delete(sums[0], j, 0), j, 1)
    assert np.all(np.isfinite(finite)) and np.array_equal(finite, np.delete(np.delete(sums[2], j, 0), j, 1))
