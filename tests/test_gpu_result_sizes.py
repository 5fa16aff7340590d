"""CountsPipeline.result() hands out the device arrays on either side of the size up to which
they are copied together, as arrays of their own."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K", [1, 32768, 32769, 65536])
def test_result_is_the_device_arrays(K):
    import paper_2503_12749_amd as mp
    p = mp.CountsPipeline(0.8 * np.eye(3, dtype=complex), np.full(3, 0.5), prec="fp64", seed=2, d=1,
                          mode="joint", windows=[(0, K)], n_sub=2, samples_per_sub=4, chunk=8)
    p.run(8)
    got = p.result()
    for a, b in zip(got, (p.P_re, p.P_im, p.sigma)):
        assert a.dtype == np.float64 and a.shape == (K,) and np.array_equal(a, b.cpu().numpy())
    kept = [a.copy() for a in got]
    got[0][:] = 7.0  # none is a view of another
    assert np.array_equal(got[1], kept[1]) and np.array_equal(got[2], kept[2])
    p.P_im[K - 1] = np.nan
    with pytest.raises(mp.MPError):
        p.result()
