"""FP32 pair sums at the edges of the sample slabs (32 samples): sub-ensembles
of one sample, of one slab less one, one slab, one more, two stages and a tail, and
chunks that cut them, on two 128-mode tiles (one diagonal pair of each kind and one
off-diagonal pair).  Oracle and tolerance are the pair-moment test's: twice the
first-order propagation bound plus 4 K u of the sum of magnitudes over a
sub-ensemble's K samples."""
import numpy as np
import pytest

from oracle import estimator as oest
from oracle import sampler as osamp
from test_gpu_pairs import DEV, _network, _tolerance

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ns,chunk", [(1, 4), (31, 124), (32, 50), (33, 132), (65, 97), (129, 260)])
def test_pair_sums_at_slab_edges(ns, chunk):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2503_12749_amd as mp
    M, n_sub, seed = 130, 4, 23
    E = ns * n_sub
    T = _network(M, 7)
    r = np.linspace(0.4, 1.1, M)
    p = mp.PairPipeline(T, r, prec="fp32", seed=seed, n_sub=n_sub, samples_per_sub=ns, chunk=chunk,
                        device=DEV)
    p.run()
    got = p.subensemble_sums()
    ref = oest.pair_correlations(T, r, seed, E, n_sub, chunk=chunk)
    a, b, _ = osamp.sample(r, 0, E, seed)
    ap, bp = oest.propagate(T, a, b)
    for s in range(n_sub):
        sl = slice(s * ns, (s + 1) * ns)
        tol = _tolerance("fp32", a[sl], b[sl], ap[sl], bp[sl])
        assert np.all(np.abs(got[s] - ref["Ps"][s] * ns) <= tol), s
