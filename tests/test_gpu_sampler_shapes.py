"""The sampler at the edges of its kernels (lanes per sample in small networks,
samples per wave and workgroup, blocks of mode pairs held in LDS, odd chunks)
against the oracle's draws."""
import numpy as np
import pytest

from oracle import sampler as osampler

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp64", "fp32", "split1t_fp16"])
@pytest.mark.parametrize("M,E", [(1, 70), (2, 33), (3, 1), (5, 65), (33, 17), (63, 40), (64, 21),
                                 (65, 19), (127, 16), (2049, 7), (4100, 3)])
def test_stored_amplitudes(prec, M, E):
    import torch

    import paper_2503_12749_amd as mp
    r = np.random.default_rng(M).uniform(0.2, 1.3, M)
    seed, net, g0 = 77, 3, 2 ** 40 + 5
    p = mp.CountsPipeline(np.eye(M, dtype=complex), r, prec=prec, seed=seed, net=net, windows=[(0, 4)],
                          n_sub=1, samples_per_sub=E, chunk=E)
    p.ab.fill_(0xFF)  # whatever is not written would show
    mp.mp_sample(M, g0, E, p.r, seed, net, p.prec, p.ab, p.n)
    torch.cuda.synchronize()
    a, b = p.alpha_beta(E)
    ra, rb = osampler.sample(r, g0, E, seed, net)[:2]
    # FP64: a few ulps of the terms; FP32: the roundings of the coefficients, the radius, the
    # sine and cosine and the FMA (6 u of c+ |w1| + c- |w2|, at most 5 (c+ + c-) here); FP16:
    # half an ulp of the value more
    top = np.sqrt(np.expm1(2 * r)) * 5
    tol = {"fp64": 1e-14, "fp32": 6 * 2.0 ** -24, "split1t_fp16": 6 * 2.0 ** -24}[prec] * top
    half = 2.0 ** -11 if prec == "split1t_fp16" else 0.0
    for got, ref in ((a, ra), (b, rb)):
        assert np.all(np.abs(got - ref) <= tol + half * np.abs(ref) + (2.0 ** -24 if half else 0))
    n = (a * b).sum(1)
    assert np.abs(p.n[:E].cpu().numpy() - n).max() <= 1e-13 * (np.abs(a * b).sum(1)).max()
    # padding modes are zero
    ldm = mp.mp_ld_modes(M)
    if prec != "split1t_fp16":
        v = p.ab.view(torch.float64 if prec == "fp64" else torch.float32)[: 2 * E * ldm]
        assert not v.view(2 * E, ldm)[:, M:].any()
    else:
        e2 = E + (E & 1)
        v = p.ab.view(torch.float16)[: 2 * e2 * ldm].view(e2, ldm // 32, 2, 32).permute(0, 2, 1, 3)
        v = v.reshape(2 * e2, ldm)
        assert not v[:, M:].any() and not v[E:e2].any() and not v[e2 + E:].any()


@pytest.mark.parametrize("prec", ["split_bf16", "split_fp16", "split1t_f8"])
def test_small_and_large_paths_agree(prec):
    """A network of 64 modes (several samples per wave) stores what the first 64 modes of one of
    65 modes (a sample per wave) do."""
    import torch

    import paper_2503_12749_amd as mp
    E, rows = 37, []
    r = torch.linspace(0.3, 1.2, 65, dtype=torch.float64, device="cuda")
    for M in (64, 65):
        ab = torch.full((mp.mp_ab_bytes(M, E, prec),), 0xFF, dtype=torch.uint8, device="cuda")
        n = torch.empty(E, dtype=torch.float64, device="cuda")
        mp.mp_sample(M, 9, E, r, 5, 0, prec, ab, n)
        rows.append(ab.cpu().numpy())
    # mode 64 is the first value of the third (second) 32 (64) mode block of its column
    x, y = rows[0].copy(), rows[1].copy()
    assert x.size == y.size
    differ = np.flatnonzero(x != y)
    cols = 2 * (E + (E & 1) if prec == "split1t_f8" else E)
    if prec == "split1t_f8":
        fp16, f8 = differ[differ < 4 * (cols // 2) * 128], differ[differ >= 4 * (cols // 2) * 128]
        f8 = f8 - 4 * (cols // 2) * 128
        assert np.all((fp16 % 512) // 128 == 2) and np.all((fp16 % 64) < 2)
        assert np.all((f8 % 256) // 128 == 1) and np.all(f8 % 64 == 0)
    else:
        assert np.all((differ % 512) // 128 == 2) and np.all(differ % 64 < 2)
