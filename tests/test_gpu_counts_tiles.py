"""The counting kernel at the edges of its tiles: samples per workgroup, grid
points listed at a time, bins and runs, against the generating function summed
in numpy."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _sums(occ, n, windows, e0, ns, n_sub, plus_p):
    """occ: list of complex (E,) occupations, one per distribution.  Sums of chi and of its
    terms' magnitudes on the concatenated grids, per sub-ensemble."""
    sub = (e0 + np.arange(len(n))) // ns
    L = np.log1p(np.exp(-2 * np.abs(n)))
    c = [np.zeros_like(n)] if plus_p else [np.minimum(2 * n, 0) - L, np.minimum(-2 * n, 0) - L]
    acc, mag = [], []
    for v, (lo, K) in zip(occ, windows):
        k = np.arange(K)
        th = 2 * np.pi * k / K
        shift = -2j * np.pi * ((k * lo) % K) / K
        a, m = np.zeros((n_sub, K), complex), np.zeros((n_sub, K))
        for s in range(n_sub):
            i = sub == s
            for sign, ct in zip((1, -1), c):
                x = np.exp(sign * v[i, None] * (np.exp(1j * th) - 1) + ct[i, None] + shift)
                a[s] += x.sum(0)
                m[s] += np.abs(x).sum(0)
        acc.append(a)
        mag.append(m)
    return np.concatenate(acc, 1), np.concatenate(mag, 1)


# one sample; around the 64 of a workgroup; tiles of more than 64 (from 512 x 64 samples on);
# windows of one point, below and above the 512 threads and the 2048 points listed at a time
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("E,ns,e0,K", [(1, 1, 0, (1, 3, 5)), (65, 64, 63, (40, 7, 600)),
                                       (130, 50, 7, (2100, 64, 513)), (36000, 7001, 6000, (9, 3, 24))])
@pytest.mark.parametrize("plus_p,mean", [(False, 4.0), (False, 900.0), (True, 2.0)])
def test_counts_from_c(prec, E, ns, e0, K, plus_p, mean):
    import torch

    import paper_2503_12749_amd as mp
    rng = np.random.default_rng(E + K[0])
    n_sub = (e0 + E - 1) // ns + 1
    dt = np.float64 if prec == "fp64" else np.float32
    occ = mean + 0.1 * mean * rng.standard_normal((2, E)) + 0.2j * np.sqrt(mean) * rng.standard_normal((2, E))
    occ = occ.real.astype(dt).astype(float) + 1j * occ.imag.astype(dt).astype(float)
    n = occ.real.sum(0) * 1.05 + rng.standard_normal(E)
    # alpha' = 1, beta' = n' in modes 1 and 2 of three; mode 0 is not counted
    M, ldm = 3, mp.mp_ld_modes(3)
    C = np.zeros((2 * E, 2, ldm), dtype=dt)
    C[:, 0, 0] = 7.0
    C[:E, 0, 1:3] = 1.0
    C[E:, 0, 1:3] = occ.real.T
    C[E:, 1, 1:3] = -occ.imag.T
    win = [(3, K[0]), (0, K[1]), (5, K[2])]
    acc = torch.zeros(n_sub * sum(K) * 2, dtype=torch.float64, device="cuda")
    ws = torch.empty(mp.mp_binned_workspace(2, "marginals_and_total", K, E, n_sub, ns, e0),
                     dtype=torch.uint8, device="cuda")
    mp.mp_binned_counts(M, E, torch.from_numpy(C.reshape(-1)).cuda(), torch.from_numpy(n).cuda(), prec,
                        "plus_p" if plus_p else "matrix_p", 2, [-1, 0, 1], "marginals_and_total",
                        [w[0] for w in win], K, n_sub, ns, e0, acc, ws)
    got = acc.cpu().numpy().view(complex).reshape(n_sub, -1)
    ref, mag = _sums([occ[0], occ[1], occ.sum(0)], n, win, e0, ns, n_sub, plus_p)
    # FP32: exponents of at most 46 and phases within pi rounded to 2^-24, the functions to a
    # few ulps; FP64: exponents and phases of up to 8 mean
    u, arg = (2.0 ** -24, 46.0) if prec == "fp32" else (2.0 ** -53, 46 + 32 * mean)
    assert np.all(np.abs(got - ref) <= 2 * (arg + 16) * u * mag + E * np.exp(-46.0))


# partials of one and several 128-mode blocks per run, more runs than bins, tiles above 64 samples
@pytest.mark.parametrize("M,E", [(130, 70), (700, 129), (300, 36001)])
def test_counts_from_partials(M, E):
    import torch

    import paper_2503_12749_amd as mp
    bins = np.full(M, -1, np.int32)
    for lo, hi, b in ((0, M // 5, 1), (M // 5, M // 2, 0), (M // 2 + 3, M, 1)):
        bins[lo:hi] = b
    K, ns = (60, 33, 128), 9001
    n_sub = -(-E // ns)
    p = mp.CountsPipeline(np.eye(M, dtype=complex), np.full(M, 0.3), prec="fp32", seed=4, bin_of_mode=bins,
                          d=2, mode="marginals_and_total", windows=[(0, k) for k in K], n_sub=n_sub,
                          samples_per_sub=ns, chunk=E, fused=True)
    p.run_chunk(0, E)
    a, b = p.alpha_beta(E)
    occ = [(a * b)[:, bins == q].sum(1) + 0j for q in range(2)]
    occ.append(occ[0] + occ[1])
    got = p.acc.cpu().numpy().view(complex).reshape(n_sub, -1)
    n = p.n[:E].cpu().numpy()
    ref, mag = _sums(occ, n, [(0, k) for k in K], 0, ns, n_sub, False)
    # T = 1: alpha', beta' are the stored amplitudes; their products sum in FP32 over 64-row
    # halves of a 128-mode block, an error of at most 64 u sum |alpha beta| in n_q, which moves
    # a term by twice that; and the terms' own rounding
    dn = 64 * 2.0 ** -24 * np.abs(a * b).sum(1).max()
    assert np.all(np.abs(got - ref) <= (4 * dn + 2 * 62 * 2.0 ** -24) * mag + E * np.exp(-46.0))
