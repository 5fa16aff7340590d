"""The surrogate's row-wise forward and backward kernels at the edges of their
tiles, against the FP64 MLP oracle."""
import ctypes

import numpy as np
import pytest

from oracle import mlp as omlp

pytestmark = pytest.mark.gpu


# one and several layers; widths that start rows on odd, even and 16-byte aligned addresses;
# 32-column and 256-column passes and their remainders, the widest layer; batches around the
# 16 rows of a workgroup and the batch quarters of the weight gradient
@pytest.mark.parametrize("width", [(3, 2), (1, 1, 1), (5, 33, 31, 8), (7, 256, 8, 257, 3),
                                   (5, 34, 130, 16, 8), (9, 1024, 1023, 6), (4, 8, 16, 24, 32, 40, 48, 56, 64)])
@pytest.mark.parametrize("batch", [1, 17, 64, 129])
def test_loss_gradients_and_forward(width, batch):
    from paper_2503_12749_amd.surrogate import Mlp
    rng = np.random.default_rng(sum(width) + batch)
    net = Mlp(width=width, batch_max=batch, seed=sum(width))
    X = rng.normal(size=(batch, width[0])).astype(np.float32)
    Y = rng.normal(size=(batch, width[-1])).astype(np.float32)
    p = net.params.cpu().numpy().astype(np.float64)
    loss, g = net.loss_grad_raw(X, Y)
    ref_loss, ref_g = omlp.loss_grad(p, width, X.astype(np.float64), Y.astype(np.float64))
    # FP32 sums of at most n terms, relative error about sqrt(n) u each with a margin of 3,
    # through the forward and the backward pass of every layer; a batch of at most 129 rows
    # adds one more sum
    u, L = 2.0 ** -24, len(width) - 1
    tol = 3 * np.sqrt(max(width) + 8) * u * (2 * L + 2)
    assert abs(loss - ref_loss) <= 2 * tol * ref_loss
    off = 0
    for l in range(L):
        n = (width[l] + 1) * width[l + 1]
        a, b = g[off: off + n], ref_g[off: off + n]
        assert np.linalg.norm(a - b) <= tol * np.linalg.norm(b) + 1e-30, l
        off += n
    pred, ref = net.predict_raw(X), omlp.forward(p, width, X.astype(np.float64))[0]
    assert np.linalg.norm(pred - ref) <= tol * np.linalg.norm(ref)


def test_weights_at_an_unaligned_address():
    """The BF16 weights may start on any 2-byte address; the products are the same values in
    the same order."""
    import torch

    from paper_2503_12749_amd import _lib, _ptr, _stream
    from paper_2503_12749_amd.surrogate import Mlp
    width, batch = (5, 64, 48, 8), 40
    net = Mlp(width=width, batch_max=batch, seed=2)
    rng = np.random.default_rng(1)
    X = torch.from_numpy(rng.normal(size=(batch, 5)).astype(np.float32)).cuda()
    Y = torch.from_numpy(rng.normal(size=(batch, 8)).astype(np.float32)).cuda()
    got = []
    for shift in (0, 1):
        w = torch.empty(net.n + 1, dtype=torch.int16, device="cuda")[shift: shift + net.n]
        w.copy_(net.w16)
        _lib.check(_lib.load().mp_mlp_loss_grad(
            ctypes.byref(net.shape), _ptr(w), _ptr(net.params), _ptr(X), _ptr(Y), batch,
            _ptr(net.grads), _ptr(net.loss), _ptr(net.ws), net.ws.numel(), _stream(None)))
        got.append((net.grads.cpu().numpy().copy(), net.loss.item()))
    assert np.array_equal(got[0][0], got[1][0]) and got[0][1] == got[1][1]
