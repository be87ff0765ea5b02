"""GPU: linear gradients of which two at a time are on the chip and a third on its way (kernels_onepass.hip), against the oracle:
every shape of a thread's rows, at sizes next to the edges of the strips, with from one to many gradients to a group of blocks."""
import numpy as np
import pytest

import oracle
from test_gpu_onepass import P, TOL, _data, _engine, _err  # noqa: F401  (P is a fixture)
from workloads import random_regular4_graph, ring_graph

pytestmark = pytest.mark.gpu

# (model, M, d): rows of a wavefront 2, 4, 6, 8, 12, 16 in 1, 2, 4 and 8 groups; from 8 MB a gradient (16 MB with 6 rows) on.  The
# last of a model's rows: whole strips, one column beyond them, odd.  (96, 32 769), (128, 16 411) and (64, 65 537) are beyond what leaves
# the pipeline enough places, and go to the kernel for one gradient at a time; (96, 32 767) and (128, 16 383) are not.
SHAPES = [("logreg", 2, 1_000_003), ("logreg", 3, 699_999), ("lsq", 4, 524_289), ("lsq", 6, 699_999), ("lsq", 8, 262_144), ("lsq", 7, 300_001),
          ("logreg", 8, 1_048_573), ("lsq", 11, 400_002), ("logreg", 16, 131_075), ("lsq", 21, 200_003), ("logreg", 32, 65_541), ("lsq", 45, 100_001),
          ("lsq", 64, 40_003), ("logreg", 90, 30_017), ("lsq", 96, 32_769), ("logreg", 128, 16_411), ("lsq", 127, 65_533),
          ("lsq", 96, 32_767), ("logreg", 128, 16_383), ("logreg", 64, 65_537)]


@pytest.mark.parametrize("model,M,d", SHAPES)
def test_events(P, model, M, d):  # noqa: F811
    print("pipeline, events %s M=%d d=%d" % (model, M, d), flush=True)
    n, T, K, rows = 5, 3, 14, max(M // 2, 4)
    g = ring_graph(n)
    feats, targs = _data(model, n, rows, d)
    sched = oracle.make_schedule(g, K, seed=6, T_max=T, M=M, rows=[rows] * n)
    x0 = np.random.default_rng(3).standard_normal((n, d)).astype(np.float32)
    wait_free = M % 2 == 1 or M < 6
    Xr = x0.copy()
    r = oracle.run_events(Xr, sched, oracle.MODEL_LOGREG if model == "logreg" else oracle.MODEL_LSQ, 0.3, M=M, gscale=1.0 / M,
                          lam=1e-3 if model == "logreg" else 0.0, features=feats, targets=targs, want_loss=True, local_compensation=wait_free)
    got = []
    for limit in (None, 0):                 # 0: every block leaves the exchange at once, the gradients go in shares
        eng = _engine(P, model, g, d, M, T, feats, targs, local_compensation=wait_free)
        if limit is not None:
            eng.h.set_wait_limits(limit)
        eng.set_models(x0, broadcast=False)
        eng.run_events(sched, want_loss=True)
        assert _err(eng.get_models(), Xr) <= TOL, limit
        assert np.allclose(eng.get_loss(), r["loss"], rtol=2e-5, atol=1e-6), limit
        assert not eng.X[:, d:].any()
        assert (eng.h.get_late_blocks() > 0) == (limit == 0)
        got.append((eng.get_models(), eng.get_loss()))
        eng.close()
    assert np.array_equal(got[0][0], got[1][0]) and np.array_equal(got[0][1], got[1][1])      # the sums in the same order


# all n gradients of an iteration in one launch: n / groups of blocks each, twice with the words of the launch before.  Those that the
# kernel for one gradient at a time takes in one step go there (n = 5, 7; and 128 x 16 411, see above).  The last two are beyond the pipeline: one gradient in registers, part of the next one's rows in LDS, six and five to the one group of blocks
@pytest.mark.parametrize("want_loss", [True, False])
@pytest.mark.parametrize("model,M,d,n", [("logreg", 128, 16_411, 3), ("lsq", 128, 16_411, 4), ("logreg", 8, 262_147, 7), ("lsq", 8, 1_000_003, 9),
                                         ("lsq", 32, 65_541, 16), ("logreg", 128, 16_383, 5),
                                         ("logreg", 128, 16_383, 9), ("logreg", 8, 262_147, 3), ("lsq", 8, 262_147, 16),
                                         ("logreg", 64, 140_003, 5), ("lsq", 16, 600_001, 6), ("logreg", 128, 70_001, 5)])
def test_synchronous_iterations(P, model, M, d, n, want_loss):  # noqa: F811
    print("pipeline, synchronous %s M=%d d=%d n=%d loss=%s" % (model, M, d, n, want_loss), flush=True)
    S, rows = 3, max(M // 4, 4)
    g = ring_graph(n) if n < 6 else random_regular4_graph(n, 2)
    feats, targs = _data(model, n, rows, d)
    batch = np.random.default_rng(5).integers(0, rows, size=(S, n, M)).astype(np.int32)
    x0 = np.random.default_rng(3).standard_normal((n, d)).astype(np.float32)
    eng = _engine(P, model, g, d, M, 0, feats, targs)
    eng.set_models(x0, broadcast=False)
    eng.run_sync_steps(S, batch, want_loss=want_loss)
    Xr = x0.copy()
    r = oracle.run_sync_steps(Xr, batch, oracle.metropolis_weights(g), oracle.MODEL_LOGREG if model == "logreg" else oracle.MODEL_LSQ, 0.3, M=M,
                              gscale=1.0 / M, lam=1e-3 if model == "logreg" else 0.0, features=feats, targets=targs, steps=S, want_loss=True)
    assert _err(eng.get_models(), Xr) <= TOL
    assert not want_loss or np.allclose(eng.get_loss().reshape(-1), np.asarray(r["loss"]).reshape(-1), rtol=2e-5, atol=1e-6)
    assert eng.get_stats()["grad_launches"] == S and eng.h.get_late_blocks() == 0
    eng.close()
