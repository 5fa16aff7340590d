"""Split-precision products in tiles of 256 x 128 and of 256 x 256, on either side of the rule
between them and with ragged last tiles of 128 columns: every propagated amplitude against numpy on
the stored operands, and the counts of the stored and of the occupation-fused product against the
generating function summed in numpy on those amplitudes.

Tolerances.  Amplitudes: T keeps 2^-18 (BF16 pairs) or 2^-22 (FP16 pairs) of an element and the
dropped product of the low parts is as large, 2^-11 with one FP16 value; 3 M products are added in
FP32, whose rounding errors are taken as independent, 6 sqrt(3 M + 8) u; all relative to the norms
of the row and of the sample, twice for the two parts.  Counts: the fused product adds 64 rows of
alpha'_j beta'_j in FP32 and the halves in FP64, 72 u of the sum of magnitudes in n_q, which moves a
term by twice that for each of its two factors; a term's own exponent of at most 46 and phase
are rounded to u."""
import numpy as np
import pytest

from test_gpu_counts_tiles import _sums

pytestmark = pytest.mark.gpu

U = 2.0 ** -24


def _stored(p, prec, E):
    """(alpha, beta) as stored: (E, M) each."""
    import torch

    import paper_2503_12749_amd as mp
    if prec.startswith("split1t"):
        return p.alpha_beta(E)
    ldm = mp.mp_ld_modes(p.M)
    t = p.ab.view(torch.bfloat16 if prec == "split_bf16" else torch.float16)[: 4 * E * ldm]
    v = t.view(2 * E, ldm // 32, 2, 32).double().sum(2).reshape(2 * E, ldm)[:, : p.M].cpu().numpy()
    return v[:E], v[E:]


# one turn of narrow tiles; three narrow turns against two wide ones; two against one (wide)
@pytest.mark.parametrize("prec", ["split_bf16", "split_fp16", "split1_fp16", "split1t_fp16"])
@pytest.mark.parametrize("M,E", [(3, 1), (100, 129), (130, 65), (300, 1000), (520, 1601), (436, 10001),
                                 (300, 7001), (900, 2049)])
def test_products_and_counts(prec, M, E):
    import torch

    import paper_2503_12749_amd as mp
    rng = np.random.default_rng(M + E)
    T = (rng.standard_normal((M, M)) + 1j * rng.standard_normal((M, M))) / np.sqrt(2 * M) * 0.7
    win, accs = [(0, 24)], []
    for fused in (False, True):
        p = mp.CountsPipeline(T, np.linspace(0.2, 0.5, M), prec=prec, seed=3, d=1, mode="joint",
                              bin_of_mode=np.zeros(M, np.int32), windows=win, n_sub=1,
                              samples_per_sub=E, chunk=E, fused=fused)
        if not fused:
            p.C.fill_(255)  # NaN
        p.ws_counts.fill_(255)
        p.run_chunk(0, E)
        torch.cuda.synchronize()
        accs.append(p.acc.cpu().numpy().view(complex).reshape(1, -1))
        if fused:
            continue
        a, b = _stored(p, prec, E)
        ga, gb = p.propagated(E)
        kept = {"split_bf16": 2 * 2.0 ** -18, "split1_fp16": 2.0 ** -11}.get(prec, 2 * 2.0 ** -22)
        tol = 2 * (kept + 6 * np.sqrt(3 * M + 8) * U) * np.linalg.norm(T, axis=1)
        for x, got, want in ((a, ga, a @ T.T), (b, gb, b @ T.conj().T)):
            assert np.all(np.abs(got - want) <= np.linalg.norm(x, axis=1)[:, None] * tol)
        occ, dn = (ga * gb).sum(1), 72 * U * np.abs(ga * gb).sum(1).max()
        ref, mag = _sums([occ], p.n[:E].cpu().numpy(), win, 0, E, 1, False)
    bound = (4 * dn + 2 * 62 * U) * mag + E * np.exp(-46.0)
    assert bound.max() < 1e-2 * np.abs(ref).max()  # a missing or doubled tile would show
    for acc in accs:
        assert np.all(np.abs(acc - ref) <= bound)
