"""GPU: the divergence check at the edges of its tiles (1024, 2048 and 8192 entries of a row) against a count on the host."""
import numpy as np
import pytest

from workloads import ring_graph

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,d", [(2, 1), (3, 5), (6, 1024), (6, 1025), (5, 2048), (5, 2049), (4, 8191), (5, 8192), (3, 8193), (64, 700), (7, 40_003)])
def test_count_of_entries_that_are_not_finite(n, d):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1710_06952_amd as P
    print("count n=%d d=%d" % (n, d), flush=True)
    rng = np.random.default_rng(n * 100_003 + d)
    x = rng.standard_normal((n, d)).astype(np.float32)
    at = rng.random((n, d)) < 0.01
    x[at] = rng.choice(np.array([np.nan, np.inf, -np.inf, np.finfo(np.float32).max, np.float32(1e-45)], np.float32), size=int(at.sum()))
    x[0, 0], x[-1, -1] = np.inf, np.nan          # the first and the last entry of the models
    eng = P.Engine(ring_graph(n), d, "synth", gamma=0.1, T_max=1, synth_std=0.1, synth_seed=1)
    eng.set_models(x, broadcast=False)
    assert eng.count_nonfinite() == int(np.count_nonzero(~np.isfinite(x)))
    eng.close()
