"""GPU: least squares that overflows.  The strip kernel's blocks hold 256 columns, of which the last ones lie beyond d: an
infinite coefficient times their zeros must not reach a dot product, so the models hold what the rounds and plain numpy
give, infinities and NaN in the same places."""
import numpy as np
import pytest

from workloads import ring_graph

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [5, 300, 2060])
def test_infinities_stay_in_their_columns(d):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1710_06952_amd as P
    print("overflow d=%d" % d, flush=True)
    n, M, K, gamma = 4, 2, 24, np.float32(1.0)
    rng = np.random.default_rng(d)
    # all features positive: a gradient beyond the largest number is +inf in every column, and its step -inf; the products
    # that meet it afterwards are infinite and not NaN
    feats = [(0.5 + rng.random((8, d))).astype(np.float32) for _ in range(n)]
    targs = [np.zeros(8, np.float32) for _ in range(n)]
    k = np.arange(K)
    sched = {"worker": (k % n).astype(np.int32), "neighbour": (k % n).astype(np.int32), "tau": np.zeros(K, np.int32),      # no averaging
             "batch_idx": rng.integers(0, 8, size=(K, M)).astype(np.int32)}
    x0 = np.full((n, d), 1e37, np.float32)
    out = []
    for rounds in (False, True):
        eng = P.Engine(ring_graph(n), d, "lsq", M=M, gamma=float(gamma), T_max=0, rounds=rounds)
        eng.load_data(feats, targs)
        eng.set_models(x0, broadcast=False)
        eng.run_events(sched, want_loss=True)
        assert (eng.get_stats()["fused_launches"] == 1) == (not rounds)
        out.append((eng.get_models(), eng.get_loss(), eng.count_nonfinite(), bool(eng.X[:, d:].any())))
        eng.close()
    X = x0.copy()
    loss = np.empty(K, np.float32)
    with np.errstate(all="ignore"):
        for e in range(K):
            i = e % n
            A = feats[i][sched["batch_idx"][e]]
            r = (A * X[i]).sum(axis=1, dtype=np.float32)
            loss[e] = (np.float32(0.5) * r * r).sum(dtype=np.float32) / np.float32(M)
            g = ((r / np.float32(M))[:, None] * A).sum(axis=0, dtype=np.float32)
            X[i] = (X[i] + X[i]) * np.float32(0.5) - gamma * g      # the average with itself may overflow, too
    assert np.isinf(loss).any() and np.isnan(loss).any()
    for x, lo, bad, padding in out:
        assert not padding and bad == np.count_nonzero(~np.isfinite(x))
        for a, b in ((x, X), (lo, loss)):
            assert np.array_equal(np.isnan(a), np.isnan(b)) and np.array_equal(np.isposinf(a), np.isposinf(b)) and np.array_equal(np.isneginf(a), np.isneginf(b))
