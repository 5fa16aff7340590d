"""Histograms and moments on either side of their launch rules: sub-ensembles of one sample and
of a few (a sample per thread, workgroups of 64 threads), around the lengths from which
workgroups count in LDS, more than 512 workgroups, bins that do not fit with several samples per
thread, against numpy.  Observable, exactness and tolerance as in test_gpu_sample_stats."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("E,ns", [(700, 1), (5000, 767), (5000, 768), (140000, 511), (140000, 800),
                                  (530000, 2047), (530000, 2048), (600000, 300000)])
@pytest.mark.parametrize("n_bins", [7, 4094, 4095])
def test_histogram_rules(E, ns, n_bins):
    import torch

    import paper_2503_12749_amd as mp
    if E // ns > 650 and n_bins > 7:
        n_bins = 40
    rng = np.random.default_rng(E + ns + n_bins)
    e0 = 2 * ns // 3
    n_sub = (e0 + E - 1) // ns + 1
    bins = rng.integers(0, n_bins + 2, E)
    lo, width = 0.25, 1.0 / n_bins
    nq = np.zeros((E, 2))
    nq[:, 0] = -np.log(np.where(bins == 0, 0.1, np.where(bins == n_bins + 1, 2.0, lo + (bins - 0.5) * width)))
    hist = torch.zeros(n_sub * (n_bins + 2), dtype=torch.float64, device="cuda")
    n = torch.zeros(E, dtype=torch.float64, device="cuda")
    mp.mp_observable_histogram(E, n, torch.from_numpy(nq.reshape(-1)).cuda(), 1, 0, 0, "plus_p", lo, width,
                               n_bins, n_sub, ns, e0, hist)
    want = np.zeros((n_sub, n_bins + 2))
    np.add.at(want, ((e0 + np.arange(E)) // ns, bins), 1.0)
    assert np.array_equal(hist.cpu().numpy().reshape(n_sub, -1), want)


@pytest.mark.parametrize("E,ns,nd", [(300, 1, 3), (2000, 64, 1), (2000, 257, 1), (4096, 1024, 1),
                                     (4200, 4097, 2), (60000, 300, 3), (520000, 9000, 9)])
def test_moment_rules(E, ns, nd):
    import torch

    import paper_2503_12749_amd as mp
    rng = np.random.default_rng(E + ns)
    e0, kmax = ns // 2, 3
    n_sub = (e0 + E - 1) // ns + 1
    z = rng.standard_normal((E, nd)) + 1j * rng.standard_normal((E, nd))
    n = rng.standard_normal(E)
    acc = torch.zeros(n_sub * nd * kmax * 2, dtype=torch.float64, device="cuda")
    nq = torch.from_numpy(np.stack([z.real, z.imag], -1).reshape(-1).copy()).cuda()
    mp.mp_moments_accumulate(E, torch.from_numpy(n).cuda(), nq, nd, kmax, "matrix_p", n_sub, ns, e0, acc)
    got = acc.cpu().numpy().view(complex).reshape(n_sub, nd, kmax)
    edges = np.concatenate([[0], np.arange(1, n_sub) * ns - e0])
    size = np.add.reduceat(np.ones(E), edges)[:, None]
    for k in range(1, kmax + 1):
        terms = z ** k * (np.tanh(n)[:, None] if k % 2 else 1.0)
        ref = np.add.reduceat(terms, edges, axis=0)
        tol = (size + 64) * 2.0 ** -53 * np.add.reduceat(np.abs(z ** k), edges, axis=0)
        assert np.all(np.abs(got[:, :, k - 1] - ref) <= tol), k
