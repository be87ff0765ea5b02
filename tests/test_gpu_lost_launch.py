"""GPU: a launch of the strip kernel whose blocks give up waiting for each other (forced from the host: they wait for no sum,
every block ends normally).  Every call that reads or advances the models reports it until set_models."""
import numpy as np
import pytest

import oracle
from workloads import logreg_data, ring_graph

pytestmark = pytest.mark.gpu


def test_a_lost_launch_is_reported_until_the_models_are_set():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1710_06952_amd as P
    print("lost launch", flush=True)
    n, d, M, K, rows = 8, 2100, 8, 80, 24
    g = ring_graph(n)
    feats, targs, _ = logreg_data(n, rows, d, seed=5)
    sched = oracle.make_schedule(g, K, seed=6, T_max=3, M=M, rows=[rows] * n)
    kw = dict(M=M, gamma=0.05, lam=1e-3, T_max=3, momentum=0.9, weight_decay=1e-3)
    eng = P.Engine(g, d, "logreg", **kw)
    eng.load_data(feats, targs)
    x0 = np.random.default_rng(3).standard_normal((n, d)).astype(np.float32)
    eng.set_models(x0, broadcast=False)
    eng.h.set_wait_limits(lose_exchange=True)
    eng.run_events(sched, want_loss=True)
    assert eng.get_stats()["fused_launches"] == 1
    torch.cuda.synchronize()
    assert np.array_equal(eng.X[:, :d].cpu().numpy(), x0)          # the blocks wrote nothing back
    out = torch.zeros(d, dtype=torch.float64, device="cuda:0")
    p = np.full(n, 1.0 / n)
    batch = np.zeros((1, n, M), np.int32)
    for name, call in (("synchronize", eng.h.synchronize), ("get_loss", eng.get_loss), ("get_models", eng.get_models),
                       ("get_momentum", eng.get_momentum), ("get_mean_model", eng.get_mean_model),
                       ("mean_model_to_device", lambda: eng.h.mean_model_to_device(out.data_ptr())),
                       ("consensus_distance", eng.consensus_distance), ("consensus_distance p", lambda: eng.consensus_distance(p)),
                       ("consensus_distance_static", lambda: eng.h.consensus_distance_static(out.data_ptr())),
                       ("count_nonfinite", eng.count_nonfinite), ("objective", eng.objective), ("objective p", lambda: eng.objective(None, p)),
                       ("classification_error", eng.classification_error), ("run_events", lambda: eng.run_events(sched)),
                       ("run_sync_steps", lambda: eng.run_sync_steps(1, batch))):
        with pytest.raises(P.AdpsgdError) as ei:
            call()
        assert ei.value.code == -5, name
    assert np.isfinite(eng.objective(x0[0]))                       # at a point of the caller's, the models are not read
    assert eng.get_stats()["events"] == K and not out.any().item()
    # set_models replaces what is lost; nothing is left of it, nor of a launch that is still under way when it is called
    eng.set_models(x0, broadcast=False)
    eng.run_events(sched)
    eng.set_models(x0, broadcast=False)
    eng.h.set_wait_limits()
    eng.run_events(sched, want_loss=True)
    Xr, Vr = x0.copy(), np.zeros_like(x0)
    r = oracle.run_events(Xr, sched, oracle.MODEL_LOGREG, 0.05, M=M, gscale=1.0 / M, lam=1e-3, features=feats, targets=targs,
                          momentum=0.9, weight_decay=1e-3, V=Vr, want_loss=True)
    assert np.allclose(eng.get_loss(), r["loss"], rtol=2e-4, atol=1e-6)
    X = eng.get_models()
    assert np.max(np.abs(X - Xr)) <= 1e-5 * np.max(np.abs(Xr))
    eng.close()
