"""GPU: gradients of the linear models in one pass over the minibatch rows, against the oracle: every shape in which a gradient
lies on the chip (rows of a wavefront, chunks of columns, row groups), at sizes next to the edges of its strips."""
import numpy as np
import pytest

import oracle
from workloads import logreg_data, lsq_data, random_regular4_graph, ring_graph

pytestmark = pytest.mark.gpu
TOL = 1e-5


@pytest.fixture(scope="module")
def P():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1710_06952_amd as pkg
    pkg.lib()
    return pkg


def _err(a, b):
    return float(np.max(np.max(np.abs(a.astype(np.float64) - b), axis=1) / np.maximum(np.max(np.abs(b), axis=1), 1e-30)))


def _engine(P, model, g, d, M, T, feats, targs, **kw):
    """An engine whose rows are padded with NaN beyond d: nothing there may count."""
    import torch
    eng = P.Engine(g, d, model, M=M, gamma=0.3, lam=1e-3 if model == "logreg" else 0.0, T_max=T, verify_plan=True, rounds=True,
                   n_slots=max(16, T + 1), **kw)
    padded = []
    for f in feats:
        t = torch.full((f.shape[0], (d + 3) // 4 * 4 + 4), float("nan"), dtype=torch.float32, device="cuda:0")
        t[:, :d] = torch.from_numpy(f).cuda()
        padded.append(t)
    eng.load_data(padded, [torch.from_numpy(t).cuda() for t in targs])
    return eng


def _data(model, n, rows, d):
    return (logreg_data if model == "logreg" else lambda n, r, d, seed: lsq_data(n, r, d, seed=seed, feature_var=1.0 / d))(n, rows, d, seed=3)[:2]


# (model, M, d): the rows a wavefront holds are 2, 4, 6, 8, 12, 16, in 1, 2, 4 and 8 groups; the columns of a strip are
# 256 x chunks x 8 / groups.  d one below, at and one beyond a whole number of strips, odd, and the largest of a shape
SHAPES = [("logreg", 1, 50_001), ("logreg", 2, 163_841), ("logreg", 2, 25_003), ("lsq", 4, 16_384), ("logreg", 3, 65_537), ("logreg", 4, 327_679),
          ("lsq", 6, 10_241), ("lsq", 6, 40_960), ("lsq", 7, 8192), ("lsq", 8, 81_921), ("lsq", 8, 163_841), ("logreg", 9, 6001),
          ("lsq", 12, 61_441), ("lsq", 13, 40_963), ("logreg", 16, 81_919), ("logreg", 17, 12_289), ("lsq", 24, 30_721), ("lsq", 32, 40_963),
          ("logreg", 33, 4097), ("lsq", 48, 25_601), ("logreg", 50, 20_481), ("lsq", 64, 5121), ("lsq", 65, 2049), ("logreg", 90, 10_239),
          ("lsq", 96, 5121), ("logreg", 97, 2051), ("lsq", 127, 10_241), ("logreg", 128, 10_753), ("lsq", 128, 131_073), ("logreg", 60, 262_147),
          ("lsq", 64, 327_681), ("lsq", 40, 300_001), ("logreg", 96, 132_001),
          ("logreg", 2, 311_299), ("logreg", 4, 200_001), ("lsq", 48, 330_001), ("lsq", 40, 400_001), ("logreg", 70, 200_003)]


@pytest.mark.parametrize("model,M,d", SHAPES)
def test_events(P, model, M, d):
    print("one pass %s M=%d d=%d" % (model, M, d), flush=True)
    n, T, rows = (3 if M * d > 8_000_000 else 5), 3, max(M // 2, 4)
    K = 8 if M * d > 8_000_000 else 24
    g = ring_graph(n)
    feats, targs = _data(model, n, rows, d)
    sched = oracle.make_schedule(g, K, seed=6, T_max=T, M=M, rows=[rows] * n)
    x0 = np.random.default_rng(3).standard_normal((n, d)).astype(np.float32)
    mu = 0.9 if M % 2 else 0.0
    wait_free = M % 3 == 0
    if model == "lsq" and not wait_free and M < 6:
        wait_free = True
    kw = dict(momentum=mu, weight_decay=1e-3 if mu else 0.0)
    Xr, Vr = x0.copy(), np.zeros_like(x0)
    r = oracle.run_events(Xr, sched, oracle.MODEL_LOGREG if model == "logreg" else oracle.MODEL_LSQ, 0.3, M=M, gscale=1.0 / M,
                          lam=1e-3 if model == "logreg" else 0.0, features=feats, targets=targs, V=Vr if mu else None, want_loss=True,
                          local_compensation=wait_free, **kw)
    got = []
    for limit in (None, 0):                 # 0: every block leaves the exchange at once, the gradients go in shares
        eng = _engine(P, model, g, d, M, T, feats, targs, local_compensation=wait_free, **kw)
        if limit is not None:
            eng.h.set_wait_limits(limit)
        eng.set_models(x0, broadcast=False)
        eng.run_events(sched, want_loss=True)
        assert _err(eng.get_models(), Xr) <= TOL, limit
        if mu:
            assert _err(eng.get_momentum(), Vr) <= TOL, limit
        assert np.allclose(eng.get_loss(), r["loss"], rtol=2e-5, atol=1e-6), limit
        assert not eng.X[:, d:].any()
        st = eng.get_stats()
        assert st["grad_launches"] <= st["rounds"]          # one launch per round that evaluates gradients
        assert (eng.h.get_late_blocks() > 0) == (limit == 0)      # nothing else on the device: the blocks find each other
        got.append((eng.get_models(), eng.get_loss()))
        eng.close()
    assert np.array_equal(got[0][0], got[1][0]) and np.array_equal(got[0][1], got[1][1])      # the sums in the same order


@pytest.mark.parametrize("model,M,d", [("lsq", 4, 100_003), ("logreg", 16, 8193), ("lsq", 128, 2053)])
def test_synchronous_iterations(P, model, M, d):
    print("one pass, synchronous %s M=%d d=%d" % (model, M, d), flush=True)
    n, S, rows = 9, 3, max(M // 2, 4)
    g = random_regular4_graph(n, 2)
    feats, targs = _data(model, n, rows, d)
    batch = np.random.default_rng(5).integers(0, rows, size=(S, n, M)).astype(np.int32)
    x0 = np.random.default_rng(3).standard_normal((n, d)).astype(np.float32)
    eng = _engine(P, model, g, d, M, 0, feats, targs)
    eng.set_models(x0, broadcast=False)
    eng.run_sync_steps(S, batch, want_loss=True)
    Xr = x0.copy()
    r = oracle.run_sync_steps(Xr, batch, oracle.metropolis_weights(g), oracle.MODEL_LOGREG if model == "logreg" else oracle.MODEL_LSQ, 0.3, M=M,
                              gscale=1.0 / M, lam=1e-3 if model == "logreg" else 0.0, features=feats, targets=targs, steps=S, want_loss=True)
    assert _err(eng.get_models(), Xr) <= TOL
    assert np.allclose(eng.get_loss().reshape(-1), np.asarray(r["loss"]).reshape(-1), rtol=2e-5, atol=1e-6)
    assert eng.get_stats()["grad_launches"] == S and eng.h.get_late_blocks() == 0
    eng.close()


@pytest.mark.parametrize("model,M,d", [("lsq", 16, 20_001), ("logreg", 128, 4099)])
def test_a_cut_schedule_gives_the_same_bits(P, model, M, d):
    """Calls that look ahead evaluate the same gradients in other rounds and groups: the same bits."""
    print("one pass, cut schedule %s M=%d d=%d" % (model, M, d), flush=True)
    n, T, rows, K = 7, 4, M, 60
    g = ring_graph(n)
    feats, targs = _data(model, n, rows, d)
    sched = oracle.make_schedule(g, K, seed=7, T_max=T, M=M, rows=[rows] * n)
    x0 = np.random.default_rng(3).standard_normal((n, d)).astype(np.float32)
    got = []
    for cuts in ([0, K], [0, 11, 12, 40, K]):
        eng = _engine(P, model, g, d, M, T, feats, targs)
        eng.set_models(x0, broadcast=False)
        for a, b in zip(cuts, cuts[1:]):
            end = min(b + T, K)
            sc = {k: sched[k][a:end] for k in ("worker", "neighbour", "tau", "batch_idx")}
            sc["lookahead"] = end - b
            eng.run_events(sc)
        got.append(eng.get_models())
        assert eng.h.get_late_blocks() == 0
        eng.close()
    assert np.array_equal(got[0], got[1])


def test_beside_a_call_in_one_launch_of_another_handle(P):
    """Compute units that another stream's work holds for milliseconds: the blocks of the one pass cannot all be there."""
    import time
    import torch
    print("one pass beside a call in one launch on another stream", flush=True)
    n, d, M, rows, K, T = 16, 65_536, 128, 128, 40, 4
    streams = [torch.cuda.Stream() for _ in range(2)]
    handles = []
    for stream, (hn, hd, hM, hrows, hK, model) in zip(streams, [(n, d, M, rows, K, "logreg"), (16, 4096, 8, 64, 16_000, "lsq")]):
        with torch.cuda.stream(stream):
            g = ring_graph(hn)
            eng = P.Engine(g, hd, model, M=hM, gamma=0.1, lam=1e-3 if model == "logreg" else 0.0, T_max=T, rounds=model == "logreg")
            eng.load_data(*_data(model, hn, hrows, hd))
            handles.append((eng, oracle.make_schedule(g, hK, seed=3, T_max=T, M=hM, rows=[hrows] * hn)))
    (eng, sched), (long, long_sched) = handles
    alone = []
    for e, s in handles * 2:
        e.set_models(np.zeros(e.d, np.float32))
        start = time.perf_counter()
        e.run_events(s)
        e.h.synchronize()
        alone.append(time.perf_counter() - start)
    ref, before = eng.get_models(), eng.h.get_late_blocks()
    eng.set_models(np.zeros(d, np.float32))
    torch.cuda.synchronize()
    start = time.perf_counter()
    long.run_events(long_sched)
    eng.run_events(sched)
    eng.h.synchronize()
    elapsed = time.perf_counter() - start
    assert before == 0 and eng.h.get_late_blocks() > 0
    assert np.array_equal(eng.get_models(), ref)
    assert elapsed <= 3 * (alone[2] + alone[3]), (elapsed, alone)          # at most one after the other, and the waits
    eng.close()
    long.close()


def test_a_handle_is_created_without_waiting_for_other_streams(P):
    import torch
    print("one pass, handle created beside work of the default stream", flush=True)
    other = torch.cuda.Stream()
    x = torch.zeros(256 << 20, device="cuda:0")
    with torch.cuda.stream(other):
        warm = P.Engine(ring_graph(40), 70_000, "logreg", M=16, gamma=0.1, T_max=2)
    torch.cuda.synchronize()
    for _ in range(600):                    # 1 GB read and written each: about 0.2 s
        x.add_(1.0)
    done = torch.cuda.Event()
    done.record()
    with torch.cuda.stream(other):
        eng = P.Engine(ring_graph(40), 70_000, "logreg", M=16, gamma=0.1, T_max=2)
    assert not done.query()
    torch.cuda.synchronize()
    eng.close()
    warm.close()
