"""Launches of more than 2^32 threads: a sampled chunk that needs them is computed to the end.  (A launch counts its threads along one dimension in 32 bits.)"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _memory(gib):
    import torch
    if torch.cuda.mem_get_info()[0] < gib * 2 ** 30:
        pytest.skip(f"needs {gib} GiB of free device memory")


# 32 lanes per sample in a network of 33 modes: more than 2^32 from 2^27 samples on
def test_sample_of_a_wide_chunk():
    import torch

    import paper_2503_12749_amd as mp
    _memory(72)
    M, E, prec, tail = 33, 2 ** 27 + 2 ** 20, "split1t_fp16", 1000
    r = torch.full((M,), 0.6, dtype=torch.float64, device="cuda")
    ab = torch.empty(mp.mp_ab_bytes(M, E, prec), dtype=torch.uint8, device="cuda")
    n = torch.full((E,), np.nan, dtype=torch.float64, device="cuda")
    mp.mp_sample(M, 0, E, r, 1, 0, prec, ab, n)
    assert bool(torch.isfinite(n).all())
    small = torch.empty(mp.mp_ab_bytes(M, tail, prec), dtype=torch.uint8, device="cuda")
    n_small = torch.empty(tail, dtype=torch.float64, device="cuda")
    mp.mp_sample(M, E - tail, tail, r, 1, 0, prec, small, n_small)
    assert torch.equal(n[E - tail:], n_small)
    bytes_of = small.numel() // 2  # alpha's columns, then beta's
    for half in range(2):
        end = (half + 1) * (ab.numel() // 2)
        assert torch.equal(ab[end - bytes_of: end], small[half * bytes_of: (half + 1) * bytes_of])
    del ab, n
    torch.cuda.empty_cache()
