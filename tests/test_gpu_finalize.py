"""Inverse DFT and sub-ensemble statistics of mp_counts_finalize on arbitrary
accumulators, against numpy's FFT in FP64."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _run(d, mode, K, n_sub, acc, ns, ws_bytes=None):
    import torch

    import paper_2503_12749_amd as mp
    entries = mp.mp_acc_entries(d, mode, K)
    dev = torch.from_numpy(np.ascontiguousarray(acc).view(np.float64).reshape(-1)).cuda()
    out = [torch.full((entries,), np.nan, dtype=torch.float64, device="cuda") for _ in range(3)]
    need = mp.mp_finalize_workspace(d, mode, K, n_sub) if ws_bytes is None else ws_bytes
    ws = torch.empty(need, dtype=torch.uint8, device="cuda") if need else None
    mp.mp_counts_finalize(d, mode, K, n_sub, ns, dev, *out, ws)
    return [o.cpu().numpy() for o in out]


def _banded(rng, n_sub, K):
    """Accumulators as the counting kernels leave them: zero outside a band around 0 and K / 2."""
    a = rng.standard_normal((n_sub, K)) + 1j * rng.standard_normal((n_sub, K))
    k = np.arange(K)
    near = np.minimum(np.minimum(k, K - k), np.abs(k - K // 2)) <= K // 7
    return a * near


def _check(P, Pi, sigma, ref, scale):
    """scale: bound of the rounding error of one sub-ensemble's value."""
    assert np.abs(P - ref.real.mean(0)).max() <= scale
    assert np.abs(Pi - ref.imag.mean(0)).max() <= scale
    if len(ref) == 1:
        assert np.all(np.isnan(sigma))
    else:
        assert np.abs(sigma - ref.real.std(0, ddof=1) / np.sqrt(len(ref))).max() <= 2 * scale


# edges of the 16-point output tile, of the 32 phases of the frequency sum, of the 512 terms
# staged at a time, of the 64-entry twiddle table, and of the groups of at most 6 sub-ensembles
@pytest.mark.parametrize("K", [1, 2, 15, 17, 31, 33, 511, 513, 1025, 4160])
@pytest.mark.parametrize("n_sub", [1, 6, 13])
def test_one_distribution(K, n_sub):
    rng = np.random.default_rng(K * 100 + n_sub)
    a, ns = _banded(rng, n_sub, K), 37
    ref = np.fft.fft(a, axis=1) / (K * ns)
    # per term: a twiddle within 8 roundings (two table entries and their product), the FMA
    # chain of its phase (2 per term, K / 32 terms) and the sum of the 32 phases
    scale = 2.0 ** -53 * (8 + 32 + K / 16) * np.abs(a).sum(1).max() / (K * ns) + 1e-300
    _check(*_run(1, "joint", [K], n_sub, a, ns), ref, scale)


def test_largest_window_and_marginals():
    rng = np.random.default_rng(5)
    K, n_sub, ns = [65536, 100, 33], 2, 3
    a = np.concatenate([_banded(rng, n_sub, k) for k in K], axis=1)
    P, Pi, sigma = _run(2, "marginals_and_total", K, n_sub, a, ns)
    at = np.cumsum([0] + K)
    for k, lo, hi in zip(K, at, at[1:]):
        ref = np.fft.fft(a[:, lo:hi], axis=1) / (k * ns)
        scale = 2.0 ** -53 * (8 + 32 + k / 16) * np.abs(a[:, lo:hi]).sum(1).max() / (k * ns)
        _check(P[lo:hi], Pi[lo:hi], sigma[lo:hi], ref, scale)


# lines with and without a factorisation (primes, 2 x prime, 16 x 16 and more), several lines
# per workgroup with a remainder, the longest line, one point; each with the least workspace
# (one sub-ensemble per launch) and with the queried one
@pytest.mark.parametrize("K", [(1, 1), (7, 1), (16, 16), (17, 64), (100, 257), (3, 4093), (4096, 2),
                               (1024, 48), (128, 96, 5), (33, 16, 130), (1, 1, 9), (12, 10, 8, 6)])
@pytest.mark.parametrize("n_sub", [1, 5])
def test_joint_grid(K, n_sub):
    import paper_2503_12749_amd as mp
    d, ns = len(K), 11
    rng = np.random.default_rng(sum(K) * 10 + n_sub)
    cells = int(np.prod(K))
    a = rng.standard_normal((n_sub,) + K) + 1j * rng.standard_normal((n_sub,) + K)
    for b, k in enumerate(K):  # zero outside a box
        i = np.arange(k)
        keep = (np.minimum(i, k - i) <= k // 3).reshape([-1 if q == b + 1 else 1 for q in range(d + 1)])
        a = a * keep
    ref = (np.fft.fftn(a, axes=tuple(range(1, d + 1))) / (cells * ns)).reshape(n_sub, -1)
    # per axis: twiddle chains of 16 and 8 rotations (4 roundings each) and two sums of at
    # most 16 and K terms
    scale = 2.0 ** -53 * sum(64 + 32 + 16 + k for k in K) * np.abs(a).reshape(n_sub, -1).sum(1).max()
    scale /= cells * ns
    out = []
    for ws in (mp.mp_finalize_workspace(d, "joint", K, 1), None):
        out.append(_run(d, "joint", K, n_sub, a, ns, ws))
        _check(*out[-1], ref, scale)
    for x, y in zip(*out):
        assert np.array_equal(x, y, equal_nan=True)
