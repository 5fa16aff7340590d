"""Sums of three- and four-bin generating functions (mp_binned_counts, MP_JOINT) of
chosen bin occupations, at the edges of the row and column tiles (128 box points, 64 in
FP64), their 32-point blocks and the slabs of 32 samples, with occupations that reach all,
some or few of the blocks, against numpy."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _sums(occ, n, K, m_lo, e0, ns, n_sub, plus_p):
    """(sums of chi, sums of the magnitudes of its terms) on the grid, per sub-ensemble."""
    d = len(K)
    acc = np.zeros((n_sub,) + K, dtype=np.complex128)
    mag = np.zeros((n_sub,) + K)
    th = [2 * np.pi * np.arange(k) / k for k in K]
    shift = [np.exp(-2j * np.pi * ((np.arange(k) * lo) % k) / k) for k, lo in zip(K, m_lo)]
    L = np.log1p(np.exp(-2 * np.abs(n)))
    c = [np.zeros_like(n)] if plus_p else [np.minimum(2 * n, 0) - L, np.minimum(-2 * n, 0) - L]
    for i in range(len(n)):
        for sign, ct in zip((1, -1), c):
            x = np.ones(1)
            for b in range(d):
                f = np.exp(sign * occ[b, i] * (np.exp(1j * th[b]) - 1) + ct[i] / d) * shift[b]
                x = np.multiply.outer(x, f)
            acc[(e0 + i) // ns] += x[0]
            mag[(e0 + i) // ns] += np.abs(x[0])
    return acc, mag


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("plus_p", [False, True])
@pytest.mark.parametrize("K,mean", [((3, 5, 7), 1.0), ((9, 33, 65), 3.0), ((5, 128, 128), 25.0),
                                    ((11, 67, 131), 40.0), ((40, 21, 257), 9.0),
                                    ((3, 4, 5, 6), 1.0), ((7, 6, 40, 129), 12.0)])
def test_jointd_sums(prec, plus_p, K, mean):
    import torch

    import paper_2503_12749_amd as mp
    d = len(K)
    rng = np.random.default_rng(int(10 * mean) + K[1])
    E, e0, ns, n_sub, m_lo = 77, 13, 33, 3, (3, 0, 7, 1)[:d]
    occ = mean * (0.4 + 1.2 * rng.random((d, E))) + 0.3j * np.sqrt(mean) * rng.standard_normal((d, E))
    n = occ.real.sum(0) * 1.1 + rng.standard_normal(E)
    dt = np.float64 if prec == "fp64" else np.float32
    occ = (occ.real.astype(dt) + 1j * occ.imag.astype(dt)).astype(np.complex128)
    # alpha' = 1 and beta' = n' in the modes of the bins
    ldm = mp.mp_ld_modes(d)
    C = np.zeros((2 * E, 2, ldm), dtype=dt)
    C[:E, 0, :d] = 1.0
    C[E:, 0, :d] = occ.real.T
    C[E:, 1, :d] = -occ.imag.T
    acc = torch.zeros(n_sub * int(np.prod(K)) * 2, dtype=torch.float64, device="cuda")
    ws = torch.empty(mp.mp_binned_workspace(d, "joint", K, E, n_sub, ns, e0), dtype=torch.uint8,
                     device="cuda")
    mp.mp_binned_counts(d, E, torch.from_numpy(C.reshape(-1)).cuda(), torch.from_numpy(n).cuda(), prec,
                        "plus_p" if plus_p else "matrix_p", d, list(range(d)), "joint", m_lo, K, n_sub,
                        ns, e0, acc, ws)
    got = acc.cpu().numpy().view(np.complex128).reshape((n_sub,) + K)
    ref, mag = _sums(occ, n, K, m_lo, e0, ns, n_sub, plus_p)
    # FP32: each factor's exponent (at most about 46 + 2 |n_b| where it matters) is rounded to
    # 2^-24 relative, its phase (within pi) and its parts to a few 2^-24, and a sub-ensemble's sums
    # to 2 ns 2^-24; FP64: the same in 2^-53 with phases up to 2 |n_b| + 2 pi; terms left out are
    # below e^-46 each
    u, arg = (2.0 ** -24, 46 + 2 * mean) if prec == "fp32" else (2.0 ** -53, 46 + 8 * mean)
    bound = (d * (arg + 16) + 2 * ns) * u * mag + E * np.exp(-46.0)
    bad = np.abs(got - ref) > bound
    assert not bad.any(), (np.argwhere(bad)[:4], np.abs(got - ref)[bad][:4], bound[bad][:4])
