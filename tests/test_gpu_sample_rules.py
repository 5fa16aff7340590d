"""Moments on either side of their launch rule: sub-ensembles of one sample and of a few
(workgroups of 64 threads), of many, and more than 512 workgroups, against numpy.  Tolerance as
in test_gpu_sample_stats."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


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
