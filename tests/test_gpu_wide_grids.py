"""Launches of more than 2^32 threads: a sampled chunk and a training batch that need them are
computed to the end.  (A launch counts its threads along one dimension in 32 bits.)"""
import ctypes

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


# 32 threads per row of the batch: more than 2^32 from 2^27 rows on
def test_gradients_of_a_wide_batch():
    import torch

    from paper_2503_12749_amd import _lib, _ptr, _stream
    from paper_2503_12749_amd.surrogate import Mlp
    _memory(8)
    batch, tail = 2 ** 27 + 100, 1000
    net = Mlp(width=(1, 1), batch_max=batch, seed=4)
    rng = np.random.default_rng(0)
    x, y = (rng.standard_normal(tail).astype(np.float32) for _ in range(2))
    X, Y = (torch.zeros(batch, dtype=torch.float32, device="cuda") for _ in range(2))
    X[batch - tail:], Y[batch - tail:] = torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda()
    net.ws.fill_(0xFF)  # NaN where a row is left out
    _lib.check(_lib.load().mp_mlp_loss_grad(
        ctypes.byref(net.shape), _ptr(net.w16), _ptr(net.params), _ptr(X), _ptr(Y), batch,
        _ptr(net.grads), _ptr(net.loss), _ptr(net.ws), net.ws.numel(), _stream(None)))
    # z = w x with the weight in 16 bits; all other rows have z = y = 0
    w = float(net.w16.view(torch.bfloat16)[0])
    d = w * x.astype(np.float64) - y
    # FP32: a product and a difference per row, then a sum of `tail` terms and four more
    u = 2.0 ** -24
    for got, terms in ((net.loss.item(), d * d / batch), (net.grads[0].item(), 2 * d * x / batch),
                       (net.grads[1].item(), 2 * d / batch)):
        size = np.abs(terms).sum() + np.abs(w * x * x / batch).sum()
        assert abs(got - terms.sum()) <= (tail + 16) * u * size
    del X, Y, net
    torch.cuda.empty_cache()
