"""GPU: the strip kernel at the numbers of rows at which its variants end, in one group of blocks and in several, against the
oracle: points of evaluation that a wavefront takes from the state, and polls that wait for the block's own words."""
import numpy as np
import pytest

import oracle
from test_gpu_strips import P, TOL, rel_err  # noqa: F401  (P is a fixture)
from workloads import logreg_data, lsq_data, ring_graph

pytestmark = pytest.mark.gpu

# rows of a wavefront: 4, 8, 12, 16 (one wavefront a gradient), 12, 16 (two), 16, 18, 22 (three), 16, 18, 22 (six)
ROWS = [1, 4, 5, 12, 13, 17, 24, 25, 49, 54, 55, 97, 108, 109]


# the last two: 160 strips, up to which six wavefronts with up to 108 samples have 18 rows each, and 161
@pytest.mark.parametrize("M,d", [(M, d) for d in (259, 9001) for M in ROWS] + [(108, 40_960), (108, 40_961)])
def test_rows_of_a_variant(P, M, d):  # noqa: F811
    print("strip rows M=%d d=%d" % (M, d), flush=True)
    n, K, T, rows = 5, 40, 4, max(M, 24)
    model, mu, comp = ("lsq", "logreg")[M % 2], (0.0, 0.9)[M % 3 == 1], M % 3 == 0 or M % 4 == 1
    g = ring_graph(n)
    feats, targs = (lsq_data(n, rows, d, seed=5, feature_var=1.0 / d) if model == "lsq" else logreg_data(n, rows, d, seed=5))[:2]
    lam, gamma, wd = (0.0 if model == "lsq" else 1e-3), (0.03 if mu else 0.3), (1e-3 if mu else 0.0)
    sched = oracle.make_schedule(g, K, seed=6, T_max=T, M=M, rows=[rows] * n)
    x0 = np.random.default_rng(3).standard_normal((n, d)).astype(np.float32)
    eng = P.Engine(g, d, model, M=M, gamma=gamma, lam=lam, T_max=T, momentum=mu, weight_decay=wd, local_compensation=comp, verify_plan=True)
    padded = []                                   # what lies beyond d in a padded row may be anything
    import torch
    for f in feats:
        t = torch.full((rows, (d + 3) // 4 * 4), float("nan"), dtype=torch.float32, device="cuda:0")
        t[:, :d] = torch.from_numpy(f).cuda()
        padded.append(t)
    eng.load_data(padded, [torch.from_numpy(t).cuda() for t in targs])
    eng.set_models(x0, broadcast=False)
    eng.run_events(sched, want_loss=True)
    Xr, Vr = x0.copy(), np.zeros_like(x0) if mu else None
    r = oracle.run_events(Xr, sched, oracle.MODEL_LSQ if model == "lsq" else oracle.MODEL_LOGREG, gamma, M=M, gscale=1.0 / M, lam=lam,
                          features=feats, targets=targs, momentum=mu, weight_decay=wd, V=Vr, local_compensation=comp, want_loss=True)
    assert rel_err(eng.get_models(), Xr) <= TOL
    if mu:
        assert rel_err(eng.get_momentum(), Vr) <= TOL
    assert np.allclose(eng.get_loss(), r["loss"], rtol=2e-4, atol=1e-6)
    assert eng.get_stats()["rounds"] > eng.get_stats()["fused_launches"]        # in one launch
    eng.close()
