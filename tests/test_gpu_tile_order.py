"""Every tile of the propagation GEMM is computed once, whatever the numbers of row
and column tiles: one to eight row tiles, a second group of one, and column counts
around multiples of the eight XCDs' turn, against numpy on the amplitudes read back.

Tolerance: a propagated amplitude is a sum of M products, so its error is at most
2 (M + 4) u |T|_row |alpha| in FP64 (u = 2^-53) and in FP32 (2^-24, which includes T's
rounding); the FP8-corrected split keeps T to 2^-15 of each element's power of two and a missing
or doubled tile is off by the whole value, so 2^-10 is taken there."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp64", "fp32", "split1t_f8"])
@pytest.mark.parametrize("M,E", [(3, 1), (100, 129), (130, 1100), (300, 900), (520, 257),
                                 (900, 70), (1030, 1030), (1100, 128)])
def test_every_tile_once(prec, M, E):
    import torch

    import paper_2503_12749_amd as mp
    rng = np.random.default_rng(M + E)
    T = (rng.standard_normal((M, M)) + 1j * rng.standard_normal((M, M))) / np.sqrt(2 * M)
    p = mp.CountsPipeline(T, np.linspace(0.4, 0.9, M), prec=prec, seed=3, bin_of_mode=np.zeros(M, np.int32),
                          d=1, mode="joint", windows=[(0, 8)], n_sub=1, samples_per_sub=E, chunk=E)
    p.C.fill_(255)  # NaN
    p.run_chunk(0, E)
    torch.cuda.synchronize()
    a, b = p.alpha_beta(E)
    ga, gb = p.propagated(E)
    u = {"fp64": 2 * (M + 4) * 2.0 ** -53, "fp32": 2 * (M + 4) * 2.0 ** -24, "split1t_f8": 2.0 ** -10}[prec]
    rows = np.linalg.norm(T, axis=1)
    for x, got, want in ((a, ga, a @ T.T), (b, gb, b @ T.conj().T)):
        assert np.all(np.abs(got - want) <= u * np.linalg.norm(x, axis=1)[:, None] * rows)


@pytest.mark.parametrize("M,E", [(20, 32897), (70, 40000), (300, 22100)])
def test_tiles_past_the_first_turn(M, E):
    """More tiles than the persistent FP32 launch has workgroups, with ragged last columns:
    two to ten slabs per tile.  Tolerance as above."""
    import torch

    import paper_2503_12749_amd as mp
    rng = np.random.default_rng(M)
    T = (rng.standard_normal((M, M)) + 1j * rng.standard_normal((M, M))) / np.sqrt(2 * M)
    p = mp.CountsPipeline(T, np.linspace(0.4, 0.9, M), prec="fp32", seed=3, bin_of_mode=np.zeros(M, np.int32),
                          d=1, mode="joint", windows=[(0, 8)], n_sub=1, samples_per_sub=E, chunk=E)
    p.C.fill_(255)  # NaN
    p.run_chunk(0, E)
    torch.cuda.synchronize()
    a, b = p.alpha_beta(E)
    ga, gb = p.propagated(E)
    u = 2 * (M + 4) * 2.0 ** -24
    rows = np.linalg.norm(T, axis=1)
    for x, got, want in ((a, ga, a @ T.T), (b, gb, b @ T.conj().T)):
        assert np.all(np.abs(got - want) <= u * np.linalg.norm(x, axis=1)[:, None] * rows)


@pytest.mark.parametrize("prec", ["split_bf16", "split_fp16"])
@pytest.mark.parametrize("M,E", [(3, 1), (100, 65), (300, 1000), (520, 3210)])
def test_fused_and_stored_products_agree(prec, M, E):
    """Occupations from the stored product and from the fused one, in products of narrow tiles
    (one turn, or three against two).  The stored product's FP64 sums differ from the fused
    FP32 sums by at most 64 + 8 roundings of sum |alpha'_j beta'_j| per 128-mode block half,
    and so do n_q and, twice over, every term."""
    import torch

    import paper_2503_12749_amd as mp
    rng = np.random.default_rng(M + E)
    T = (rng.standard_normal((M, M)) + 1j * rng.standard_normal((M, M))) / np.sqrt(2 * M) * 0.7
    accs = []
    for fused in (False, True):
        p = mp.CountsPipeline(T, np.linspace(0.2, 0.5, M), prec=prec, seed=3, d=1, mode="joint",
                              bin_of_mode=np.zeros(M, np.int32), windows=[(0, 24)], n_sub=1,
                              samples_per_sub=E, chunk=E, fused=fused)
        p.run_chunk(0, E)
        accs.append(p.acc.cpu().numpy().view(complex))
        if not fused:
            a, b = p.propagated(E)
            dn = 72 * 2.0 ** -24 * np.abs(a * b).sum(1).max()
    # terms of at most e^(2 |n|) each lose 2 dn and FP32 roundings of exponents up to 46
    n = np.abs((a * b).sum(1))
    size = np.exp(2 * np.minimum(n, 20)).sum()
    assert np.all(np.abs(accs[0] - accs[1]) <= (4 * dn + 2 * 62 * 2.0 ** -24) * size)
