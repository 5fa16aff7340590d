"""Predictions at the edges of the forward kernel's chunks (32 inputs, 128-deep chunks,
16-deep steps) and tiles (64 x 64), against the FP64 oracle.  Tolerance: that of the forward
test of the surrogate, 1e-5 of the largest prediction (FP32 activations and sums of up to 300
products; three BF16 terms hold an activation to 2^-24)."""
import numpy as np
import pytest

from oracle import mlp as omlp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("width", [(1, 1), (5, 32, 33, 3), (31, 127, 128, 129, 8), (33, 64, 300, 65, 2),
                                   (144, 16, 112, 1)])
@pytest.mark.parametrize("batch", [1, 63, 130])
def test_forward_at_chunk_edges(width, batch):
    from paper_2503_12749_amd.surrogate import Mlp
    net = Mlp(width=width, batch_max=128, seed=2)
    X = np.random.default_rng(batch).normal(size=(batch, width[0]))
    ref, _ = omlp.forward(net.params.cpu().numpy().astype(np.float64), width,
                          X.astype(np.float32).astype(np.float64))
    np.testing.assert_allclose(net.predict_raw(X), ref, rtol=0, atol=1e-5 * np.abs(ref).max())
