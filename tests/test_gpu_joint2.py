"""Two-bin accumulation (mp_binned_counts, MP_JOINT, d = 2) of chosen bin
occupations against the generating function summed in numpy."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _sums(n1, n2, n, K, m_lo, e0, ns, n_sub, plus_p):
    """(sums of chi, sums of the magnitudes of its terms) on the grid, per sub-ensemble."""
    acc = np.zeros((n_sub,) + K, dtype=np.complex128)
    mag = np.zeros((n_sub,) + K)
    th = [2 * np.pi * np.arange(k) / k for k in K]
    shift = [np.exp(-2j * np.pi * ((np.arange(k) * lo) % k) / k) for k, lo in zip(K, m_lo)]
    L = np.log1p(np.exp(-2 * np.abs(n)))
    c = [np.zeros_like(n)] if plus_p else [np.minimum(2 * n, 0) - L, np.minimum(-2 * n, 0) - L]
    for i in range(len(n)):
        for sign, ct in zip((1, -1), c):
            f = [np.exp(sign * v[i] * (np.exp(1j * t) - 1) + ct[i] / 2) * s
                 for v, t, s in zip((n1, n2), th, shift)]
            acc[(e0 + i) // ns] += np.outer(*f)
            mag[(e0 + i) // ns] += np.abs(np.outer(*f))
    return acc, mag


# boxes that meet and that do not, windows at and around the 16-point blocks and the 16-, 32-
# and 48-point tiles, odd windows; occupations small and large
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("K,mean", [((1, 5), 1.0), ((16, 17), 3.0), ((48, 49), 8.0), ((33, 100), 20.0),
                                    ((300, 161), 250.0), ((1024, 640), 500.0)])
@pytest.mark.parametrize("plus_p", [False, True])
def test_joint2_sums(prec, K, mean, plus_p):
    import torch

    import paper_2503_12749_amd as mp
    rng = np.random.default_rng(int(10 * mean) + K[1])
    E, e0, ns, n_sub, m_lo = 151, 13, 40, 5, (3, 7)
    occ = mean + 0.1 * mean * rng.standard_normal((2, E)) + 0.2j * np.sqrt(mean) * rng.standard_normal((2, E))
    n = occ.real.sum(0) * 1.1 + rng.standard_normal(E)
    dt = np.float64 if prec == "fp64" else np.float32
    occ = (occ.real.astype(dt) + 1j * occ.imag.astype(dt)).astype(np.complex128)
    # alpha' = 1 and beta' = n' in the modes of the two bins
    M, ldm = 2, mp.mp_ld_modes(2)
    C = np.zeros((2 * E, 2, ldm), dtype=dt)
    C[:E, 0, :M] = 1.0
    C[E:, 0, :M] = occ.real.T
    C[E:, 1, :M] = -occ.imag.T
    Cd, nd = torch.from_numpy(C.reshape(-1)).cuda(), torch.from_numpy(n).cuda()
    acc = torch.zeros(n_sub * K[0] * K[1] * 2, dtype=torch.float64, device="cuda")
    ws = torch.empty(mp.mp_binned_workspace(2, "joint", K, E, n_sub, ns, e0), dtype=torch.uint8,
                     device="cuda")
    mp.mp_binned_counts(M, E, Cd, nd, prec, "plus_p" if plus_p else "matrix_p", 2, [0, 1], "joint",
                        m_lo, K, n_sub, ns, e0, acc, ws)
    got = acc.cpu().numpy().view(np.complex128).reshape((n_sub,) + K)
    ref, mag = _sums(occ[0], occ[1], n, K, m_lo, e0, ns, n_sub, plus_p)
    # FP32: each factor's exponent (at most about 46 + 2 |n_b| where it matters) is rounded to
    # 2^-24 relative, its phase (within pi) and its parts to a few 2^-24; FP64: the same in
    # 2^-53 with phases up to 2 |n_b| + 2 pi; dropped terms are below e^-46 each
    u, arg = (2.0 ** -24, 46 + 2 * mean) if prec == "fp32" else (2.0 ** -53, 46 + 8 * mean)
    bound = 2 * (arg + 16) * u * mag + E * np.exp(-46.0)
    assert np.all(np.abs(got - ref) <= bound)
