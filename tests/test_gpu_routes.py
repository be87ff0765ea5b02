"""GPU: a run of a linear model cut into calls that look ahead, where consecutive calls are executed in one launch and
round by round in turn: gradients pending across the cut are dense vectors or, from a least-squares call in rounds, the
coefficients of their minibatch rows, and every kind is applied by the route that comes next."""
import numpy as np
import pytest

import oracle
from workloads import logreg_data, lsq_data, random_extra_pairs, random_regular4_graph, ring_graph

pytestmark = pytest.mark.gpu

TOL = 1e-5          # of the whole suite for 32-bit models


def rel_err(x, ref):
    num = np.max(np.abs(x.astype(np.float64) - ref.astype(np.float64)), axis=1)
    return float(np.max(num / np.maximum(np.max(np.abs(ref.astype(np.float64)), axis=1), 1e-30)))


@pytest.mark.parametrize("first", ["auto", "rounds"])
@pytest.mark.parametrize("model,d,comp,mu", [("lsq", 4099, False, 0.0), ("lsq", 4099, False, 0.9), ("lsq", 700, True, 0.0),
                                             ("logreg", 4099, True, 0.9), ("logreg", 1030, False, 0.0)])
def test_routes_change_between_calls_that_look_ahead(model, d, comp, mu, first):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1710_06952_amd as P
    print("routes %s d=%d comp=%d mu=%g first %s" % (model, d, comp, mu, first), flush=True)
    n, K, T, M, rows = 6, 420, 5, 5, 24
    g = ring_graph(n)
    if model == "lsq":
        feats, targs, _ = lsq_data(n, rows, d, seed=4, feature_var=1.0 / d)
        omodel, gamma, lam = oracle.MODEL_LSQ, 0.03 if mu else 0.3, 0.0
    else:
        feats, targs, _ = logreg_data(n, rows, d, seed=4)
        omodel, gamma, lam = oracle.MODEL_LOGREG, 0.05 if mu else 0.5, 1e-3
    sched = oracle.make_schedule(g, K, seed=14, T_max=T, M=M, rows=[rows] * n)
    sched["gamma"] = (gamma * (1 + np.arange(K) % 2)).astype(np.float32)
    sched["extra_pairs"] = random_extra_pairs(g, sched["worker"], sched["neighbour"], max_extra=1, seed=3)
    x0 = np.random.default_rng(4).standard_normal(d).astype(np.float32)
    wd = 1e-3 if mu else 0.0
    eng = P.Engine(g, d, model, M=M, gamma=gamma, lam=lam, T_max=T, momentum=mu, weight_decay=wd, local_compensation=comp, verify_plan=True)
    eng.load_data(feats, targs)
    eng.set_models(x0)
    auto = [True, False, True, False, False, True, True] if first == "auto" else [False, True, False, True, True, False, True]
    launches = []

    def change(_done):                # after every call: what it launched, and the route of the next one
        launches.append(eng.get_stats()["fused_launches"] - sum(launches))
        eng.h.set_route(P.ROUTE_AUTO if auto[len(launches) % len(auto)] else P.ROUTE_ROUNDS)

    eng.h.set_route(P.ROUTE_AUTO if auto[0] else P.ROUTE_ROUNDS)
    eng.run_events_in_pieces(sched, 60, between=change)
    assert len(launches) == len(auto)
    if model == "lsq" and d > 2048 and not comp:      # coefficients pending from a call in rounds keep the next call on the rounds
        assert all(one or n_l > 1 for n_l, one in zip(launches, auto)), launches
        assert launches[0] == launches[2] == 1 if first == "auto" else launches[1] > 1
    else:
        assert all((n_l == 1) == one for n_l, one in zip(launches, auto)), launches
    X, V = eng.get_models(), eng.get_momentum() if mu else None
    eng.close()
    Xr = np.tile(x0, (n, 1))
    Vr = np.zeros_like(Xr) if mu else None
    extra = sched.pop("extra_pairs")
    oracle.run_events(Xr, sched, omodel, gamma, M=M, gscale=1.0 / M, lam=lam, features=feats, targets=targs, gamma_k=sched["gamma"],
                      extra_pairs=extra, momentum=mu, weight_decay=wd, V=Vr, local_compensation=comp)
    assert rel_err(X, Xr) <= TOL
    if mu:
        assert rel_err(V, Vr) <= TOL


def test_unknown_route_is_refused():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1710_06952_amd as P
    eng = P.Engine(ring_graph(4), 64, "synth", gamma=0.1, synth_std=0.1)
    with pytest.raises(P.AdpsgdError) as ei:
        eng.h.set_route(2)
    assert ei.value.code == -1
    eng.close()


# on both sides of the line, where the two routes differ by 1.3 to 2.5 times
@pytest.mark.parametrize("model,n,d,M,K,T,one", [("lsq", 8, 2000, 64, 64, 3, True), ("logreg", 8, 2000, 96, 64, 3, True), ("lsq", 8, 1024, 48, 48, 1, True),
                                                 ("lsq", 16, 65_536, 16, 12, 8, False), ("logreg", 6, 8192, 48, 16, 8, False), ("lsq", 8, 4096, 8, 2, 3, False)])
def test_route_of_short_calls(model, n, d, M, K, T, one):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1710_06952_amd as P
    print("route of a short call %s n=%d d=%d M=%d K=%d" % (model, n, d, M, K), flush=True)
    g = random_regular4_graph(n, 1) if (d, n) == (65_536, 16) else ring_graph(n)
    rows = max(M, 32)
    feats, targs, _ = lsq_data(n, rows, d, seed=5, feature_var=1.0 / d) if model == "lsq" else logreg_data(n, rows, d, seed=5)
    sched = oracle.make_schedule(g, K, seed=5, T_max=T, M=M, rows=[rows] * n)
    lam = 1e-3 if model == "logreg" else 0.0
    eng = P.Engine(g, d, model, M=M, gamma=0.1, lam=lam, T_max=T, verify_plan=True)
    eng.load_data(feats, targs)
    eng.set_models(np.zeros(d, np.float32))
    eng.run_events(sched)
    assert (eng.get_stats()["grad_launches"] == 0) == one
    ref = np.zeros((n, d), np.float32)
    oracle.run_events(ref, sched, oracle.MODEL_LSQ if model == "lsq" else oracle.MODEL_LOGREG, 0.1, M=M, gscale=1.0 / M, lam=lam, features=feats, targets=targs)
    assert rel_err(eng.get_models(), ref) <= TOL
    eng.close()
