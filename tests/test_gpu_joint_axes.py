"""The inverse DFT of joint grids on either side of its rules: one or eight outputs a thread,
first sums of one to sixteen terms (prime lengths have none), few or many lines a workgroup
and a last one that is not full, against numpy's FFT in FP64."""
import numpy as np
import pytest

from test_gpu_finalize import _check, _run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K", [(1, 1), (1, 7), (7, 1), (4, 4), (30, 5), (64, 64), (97, 89), (66, 258),
                               (254, 256), (300, 512), (512, 514), (1021, 37), (3, 2000), (5, 6, 7),
                               (24, 25, 23), (40, 36, 44), (4, 4, 500), (1, 2, 1, 3), (6, 5, 7, 9),
                               (20, 21, 22, 23)])
@pytest.mark.parametrize("n_sub", [1, 3])
def test_joint_grid(K, n_sub):
    rng = np.random.default_rng(sum(K) + n_sub)
    a = rng.standard_normal((n_sub,) + K) + 1j * rng.standard_normal((n_sub,) + K)
    if K[0] > 2:
        a[:, K[0] // 3] = 0.0  # lines of zeros, and columns that are zero in every line
    if K[-1] > 4:
        a[..., K[-1] // 2:K[-1] // 2 + 2] = 0.0
    cells, ns = int(np.prod(K)), 11
    ref = (np.fft.fftn(a, axes=range(1, len(K) + 1)) / (cells * ns)).reshape(n_sub, -1)
    # an axis adds at most K terms in two sums; a term carries a twiddle, at most 16 rotations of
    # it and another twiddle, three roundings each
    u = 2.0 ** -53 * sum(k + 3 * 18 for k in K)
    scale = u * np.abs(a).reshape(n_sub, -1).sum(1).max() / (cells * ns) + 1e-300
    _check(*_run(len(K), "joint", list(K), n_sub, a.reshape(n_sub, -1), ns), ref, scale)


@pytest.mark.parametrize("K", [(16, 24), (300, 512)])
def test_a_nan_reaches_its_sub_ensemble(K):
    rng = np.random.default_rng(K[0])
    a = rng.standard_normal(K) + 1j * rng.standard_normal(K)
    a[K[0] // 2, 3] = np.nan
    P, _, _ = _run(2, "joint", list(K), 1, a.reshape(-1), 1)
    assert np.all(np.isnan(P))
