"""Per-sample occupations at the edges of their lane groups: a row of 16 lanes per
sample (average runs up to 512 bytes) and a wave per sample (longer), runs that
start off the 16-byte boundaries, modes that no bin counts, runs of one bin apart,
and sample counts around a wave's share, against numpy.

Tolerance: 2 (m + 4) u of a run set's sum of |products| (u = 2^-53), the bound of
any order of FP64 products and sums over its m modes.  Modes outside the bins and
the padding hold NaN, which must not reach a sum."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _bins(M, runs):
    """runs: (lo, hi, bin); other modes are not counted."""
    b = np.full(M, -1, np.int32)
    for lo, hi, q in runs:
        b[lo:hi] = q
    return b


CASES = [
    (1, 1, [(0, 1, 0)]),
    (20, 5, [(1, 16, 0), (17, 20, 1)]),
    (40, 67, [(3, 20, 1), (20, 36, 0), (37, 39, 1)]),
    (131, 64, [(1, 66, 0), (66, 131, 1)]),
    (300, 17, [(0, 130, 0), (131, 195, 1), (195, 299, 2)]),
    (259, 33, [(2, 259, 0)]),
    (1100, 7, [(0, 258, 0), (259, 1099, 1)]),
    (2305, 3, [(1, 2304, 0)]),
    (90, 130, [(9 * i + 1, 9 * i + 9, i % 8) for i in range(10)]),
]


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("mode", ["marginals", "marginals_and_total"])
@pytest.mark.parametrize("M,E,runs", CASES)
def test_occupations_of_runs(prec, mode, M, E, runs):
    import torch

    import paper_2503_12749_amd as mp
    rng = np.random.default_rng(M + E)
    dt = np.float64 if prec == "fp64" else np.float32
    bins = _bins(M, runs)
    d = int(bins.max()) + 1
    ldm = mp.mp_ld_modes(M)
    C = np.full((2 * E, 2, ldm), np.nan, dtype=dt)
    C[:, :, :M] = rng.standard_normal((2 * E, 2, M)).astype(dt)
    C[:, :, :M][:, :, bins < 0] = np.nan
    n_dist = d + (mode == "marginals_and_total")
    nq = torch.full((E * n_dist * 2,), 7.0, dtype=torch.float64, device="cuda")
    mp.mp_occupations(M, E, torch.from_numpy(C.reshape(-1)).cuda(), prec, d, bins, mode, nq)
    got = nq.cpu().numpy().reshape(E, n_dist, 2)
    X = C[:, :, :M].astype(np.float64)
    a, b, c, e = X[:E, 0], X[:E, 1], X[E:, 0], X[E:, 1]
    for q in range(n_dist):
        m = bins == q if q < d else bins >= 0
        u = 2.0 * (m.sum() + 4) * 2.0 ** -53
        for comp, x, y in ((0, a * c, b * e), (1, b * c, -a * e)):
            tol = u * (np.abs(x) + np.abs(y))[:, m].sum(1)
            assert np.all(np.abs(got[:, q, comp] - (x + y)[:, m].sum(1)) <= tol), (q, comp)


@pytest.mark.parametrize("prec,M", [("fp32", 30), ("fp32", 1023), ("fp32", 1027), ("fp64", 511), ("fp64", 515)])
@pytest.mark.parametrize("E", [1, 5, 67])
def test_counts_on_both_sides_of_the_row_line(prec, M, E):
    """Two runs that start off the 16-byte boundaries, averages around 2048 bytes of each matrix
    row.  A bin sum's rounding is below the FP32 rounding of exponents and phases by far; the
    bound is the counting test's, with the bin sums' own (M u) in FP64."""
    import torch

    import paper_2503_12749_amd as mp
    from test_gpu_counts_tiles import _sums
    rng = np.random.default_rng(M + E)
    dt = np.float64 if prec == "fp64" else np.float32
    h = M // 2
    bins = _bins(M, [(1, h, 0), (h, M, 1)])
    ldm = mp.mp_ld_modes(M)
    C = np.full((2 * E, 2, ldm), np.nan, dtype=dt)
    C[:, :, :M] = (rng.standard_normal((2 * E, 2, M)) / np.sqrt(M)).astype(dt)
    C[:E, 0, :M] += dt(3 / np.sqrt(M))
    C[E:, 0, :M] += dt(3 / np.sqrt(M))
    C[:, :, 0] = np.nan
    X = C[:, :, :M].astype(np.float64)
    nj = (X[:E, 0] + 1j * X[:E, 1]) * (X[E:, 0] - 1j * X[E:, 1])
    occ = [nj[:, bins == q].sum(1) for q in range(2)]
    n = rng.uniform(2, 6, E)
    K = (40, 64)
    acc = torch.zeros(sum(K) * 2, dtype=torch.float64, device="cuda")
    ws = torch.empty(mp.mp_binned_workspace(2, "marginals", K, E, 1, E, 0), dtype=torch.uint8, device="cuda")
    mp.mp_binned_counts(M, E, torch.from_numpy(C.reshape(-1)).cuda(), torch.from_numpy(n).cuda(), prec,
                        "matrix_p", 2, bins, "marginals", (0, 0), K, 1, E, 0, acc, ws)
    ref, mag = _sums(occ, n, [(0, k) for k in K], 0, E, 1, False)
    u, arg = (2.0 ** -24, 46.0) if prec == "fp32" else (2.0 ** -53, 46 + 32 * 20 + M)
    got = acc.cpu().numpy().view(complex)
    assert np.all(np.abs(got - ref[0]) <= 2 * (arg + 16) * u * mag[0] + E * np.exp(-46.0))


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("d,M", [(2, 61), (2, 301), (3, 97), (3, 461)])
@pytest.mark.parametrize("E", [1, 6, 35])
def test_joint_sums_by_rows_and_waves(prec, d, M, E):
    """Joint sums of bins of some 30 and 150 modes (a row of lanes and a wave per sample).  The
    bound is the joint tests', with the bin sums' own (M u) in FP64."""
    import torch

    import paper_2503_12749_amd as mp
    from test_gpu_jointd_tiles import _sums
    rng = np.random.default_rng(M + E)
    dt = np.float64 if prec == "fp64" else np.float32
    w = (M - 1) // d
    bins = _bins(M, [(1 + q * w, 1 + (q + 1) * w, q) for q in range(d)])
    ldm = mp.mp_ld_modes(M)
    C = np.full((2 * E, 2, ldm), np.nan, dtype=dt)
    C[:, :, :M] = (rng.standard_normal((2 * E, 2, M)) / np.sqrt(M)).astype(dt)
    C[:, 0, :M] += dt(3 / np.sqrt(M))
    C[:, :, 0] = np.nan
    X = C[:, :, :M].astype(np.float64)
    nj = (X[:E, 0] + 1j * X[:E, 1]) * (X[E:, 0] - 1j * X[E:, 1])
    occ = np.stack([nj[:, bins == q].sum(1) for q in range(d)])
    n = occ.real.sum(0) * 1.05
    K = (12, 9, 10)[:d]
    acc = torch.zeros(int(np.prod(K)) * 2, dtype=torch.float64, device="cuda")
    ws = torch.empty(mp.mp_binned_workspace(d, "joint", K, E, 1, E, 0), dtype=torch.uint8, device="cuda")
    mp.mp_binned_counts(M, E, torch.from_numpy(C.reshape(-1)).cuda(), torch.from_numpy(n).cuda(), prec,
                        "matrix_p", d, bins, "joint", (0, 0, 0)[:d], K, 1, E, 0, acc, ws)
    ref, mag = _sums(occ, n, K, (0, 0, 0)[:d], 0, E, 1, False)
    u, arg = (2.0 ** -24, 46 + 2 * 12) if prec == "fp32" else (2.0 ** -53, 46 + 8 * 12 + M)
    got = acc.cpu().numpy().view(complex).reshape((1,) + K)
    assert np.all(np.abs(got - ref) <= (d * (arg + 16) + 2 * E) * u * mag + E * np.exp(-46.0))
