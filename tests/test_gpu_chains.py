"""GPU: updates of a round in chains (kernels_fused.hip, kernels_grad_linear.hip, kernels_mlp.hip): few workers, so that chains
are as long as they get, events without a partner, extra averaging pairs, lengths at the edges of the kernels' tiles.  The
same events one by one, or in rounds without chains, have to give the same bits."""
import numpy as np
import pytest

import oracle
from workloads import logreg_data, lsq_data, mixture_data, mlp_init, random_extra_pairs, random_regular4_graph, ring_graph, with_identity_events

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1710_06952_amd as pkg
    pkg.lib()
    return pkg


def schedule(graph, K, T, extra, **kw):
    s = oracle.make_schedule(graph, K, seed=6, T_max=T, **kw)
    s["neighbour"] = with_identity_events(s["worker"], s["neighbour"], 0.1, seed=1)
    if extra:
        s["extra_pairs"] = random_extra_pairs(graph, s["worker"], s["neighbour"], max_extra=2, seed=2)
    return s


# d: the first length that takes chains, one tile of 1024 more or less by one element, a ragged last tile
@pytest.mark.parametrize("n,d,T,mu,extra", [(3, 4097, 5, 0.0, False), (5, 5119, 0, 0.9, False), (5, 5120, 8, 0.9, False), (8, 5121, 3, 0.0, True),
                                            (12, 70_002, 16, 0.9, True)])
def test_caller_gradients_in_chains_are_the_rounds_of_the_synthetic_model(P, n, d, T, mu, extra):
    print("chains, caller's gradients n=%d d=%d T=%d mu=%g" % (n, d, T, mu), flush=True)
    K, std, wd = 200, float(np.float32(0.05)), 1e-3 if mu else 0.0
    g = random_regular4_graph(n, 3) if n >= 8 else ring_graph(n)
    sched = schedule(g, K, T, extra)
    x0 = np.random.default_rng(3).standard_normal((n, d)).astype(np.float32)
    ref = P.Engine(g, d, "synth", gamma=0.1, T_max=T, synth_std=std, synth_seed=11, momentum=mu, weight_decay=wd, rounds=True)
    ref.set_models(x0, broadcast=False)
    ref.run_events(sched)
    eng = P.Engine(g, d, "external", gamma=0.1, T_max=T, momentum=mu, weight_decay=wd, verify_plan=True)
    eng.set_models(x0, broadcast=False)

    def generator_gradient(requests, stream):
        for worker, event, xhat_ptr, g_ptr in requests:
            P.adpsgd_synth_gradient(11, event, std, d, g_ptr, stream)

    eng.h.run_events_with(sched, generator_gradient)
    assert np.array_equal(eng.get_models(), ref.get_models()) and not eng.X[:, d:].any()
    if mu:
        assert np.array_equal(eng.get_momentum(), ref.get_momentum())
    assert eng.get_stats()["rounds"] < ref.get_stats()["rounds"]
    ref.close()
    eng.close()


# in, hidden, out around the 32 x 64 tiles of the first layer and the blocks of 1024 floats behind it; dense: wait-free variant
@pytest.mark.parametrize("dims,M,mu,comp", [((32, 64, 2), 1, 0.0, False), ((40, 64, 16), 24, 0.9, False), ((64, 192, 10), 64, 0.0, False),
                                            ((72, 128, 3), 33, 0.9, False), ((24, 64, 5), 8, 0.9, True), ((32, 64, 7), 16, 0.0, True)])
def test_perceptron_in_chains_is_event_by_event(P, dims, M, mu, comp):
    print("chains, perceptron %s M=%d mu=%g comp=%d" % (dims, M, mu, comp), flush=True)
    n, rows, K = 5, 64, 60
    d = dims[0] * dims[1] + dims[1] + dims[1] * dims[2] + dims[2]
    g = ring_graph(n)
    sched = schedule(g, K, 0, False, M=M, rows=[rows] * n)
    feats, labels, _ = mixture_data(n, rows, din=dims[0], classes=dims[2], seed=9)
    out = []
    for step in (K, 1):
        eng = P.Engine(g, d, "mlp", M=M, gamma=0.05, T_max=0, mlp=dims, momentum=mu, weight_decay=1e-3 if mu else 0.0,
                       local_compensation=comp, verify_plan=True)
        eng.load_data(feats, labels)
        eng.set_models(mlp_init(*dims, seed=9))
        for k in range(0, K, step):
            eng.run_events({key: sched[key][k:k + step] for key in ("worker", "neighbour", "tau", "batch_idx")})
        out.append((eng.get_models(), eng.get_bf16_models(), eng.get_momentum() if mu else None, eng.get_stats()["rounds"]))
        eng.close()
    assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1])
    assert mu == 0.0 or np.array_equal(out[0][2], out[1][2])
    assert out[0][3] < out[1][3] == K


@pytest.mark.parametrize("model,d,M,mu,dense", [("lsq", 2049, 3, 0.0, False), ("lsq", 3076, 9, 0.9, False), ("lsq", 3077, 4, 0.9, True),
                                                ("logreg", 2051, 5, 0.0, False), ("logreg", 1023, 6, 0.9, False)])
def test_linear_models_in_chains_are_event_by_event(P, model, d, M, mu, dense):
    print("chains, %s d=%d M=%d mu=%g dense=%d" % (model, d, M, mu, dense), flush=True)
    n, rows, K = 5, 32, 80
    g = ring_graph(n)
    sched = schedule(g, K, 0, False, M=M, rows=[rows] * n)
    if model == "lsq":
        feats, targs, _ = lsq_data(n, rows, d, seed=5, feature_var=1.0 / d)
    else:
        feats, targs, _ = logreg_data(n, rows, d, seed=5)
    x0 = np.random.default_rng(3).standard_normal((n, d)).astype(np.float32)
    out = []
    for step in (K, 1):
        eng = P.Engine(g, d, model, M=M, gamma=0.05, lam=1e-3 if model == "logreg" else 0.0, T_max=0, momentum=mu,
                       weight_decay=1e-3 if mu else 0.0, dense_gradient=dense, rounds=True, verify_plan=True)
        eng.load_data(feats, targs)
        eng.set_models(x0, broadcast=False)
        for k in range(0, K, step):
            eng.run_events({key: sched[key][k:k + step] for key in ("worker", "neighbour", "tau", "batch_idx")})
        out.append((eng.get_models(), eng.get_momentum() if mu else None, eng.get_stats()["rounds"]))
        assert not eng.X[:, d:].any()
        eng.close()
    assert np.array_equal(out[0][0], out[1][0])
    assert mu == 0.0 or np.array_equal(out[0][1], out[1][1])
    assert out[0][2] < out[1][2] == K


@pytest.mark.parametrize("model,n,d,M,mu,extra", [("lsq", 16, 4096, 8, 0.0, True), ("lsq", 8, 2050, 4, 0.9, False), ("logreg", 8, 4096, 8, 0.9, False)])
def test_short_calls_of_a_handle_that_runs_in_one_launch(P, model, n, d, M, mu, extra):
    """A few events of such a handle go by rounds without chains, with the gradients of least squares as coefficients."""
    print("chains, short call %s n=%d d=%d M=%d mu=%g" % (model, n, d, M, mu), flush=True)
    rows, K = 32, 3
    g = random_regular4_graph(n, 3)
    sched = schedule(g, K, 2, extra, M=M, rows=[rows] * n)
    feats, targs, _ = lsq_data(n, rows, d, seed=5, feature_var=1.0 / d) if model == "lsq" else logreg_data(n, rows, d, seed=5)
    x0 = np.random.default_rng(3).standard_normal((n, d)).astype(np.float32)
    out = []
    for rounds in (False, True):
        eng = P.Engine(g, d, model, M=M, gamma=0.05, lam=1e-3 if model == "logreg" else 0.0, T_max=2, momentum=mu,
                       weight_decay=1e-3 if mu else 0.0, rounds=rounds, verify_plan=True)
        eng.load_data(feats, targs)
        eng.set_models(x0, broadcast=False)
        eng.run_events(sched)
        out.append((eng.get_models(), eng.get_momentum() if mu else None, eng.get_stats()["grad_launches"]))
        eng.close()
    assert out[0][2] > 0                                       # not in one launch
    assert np.array_equal(out[0][0], out[1][0]) and not np.array_equal(out[0][0], x0)
    assert mu == 0.0 or np.array_equal(out[0][1], out[1][1])


@pytest.mark.parametrize("mu", [0.0, 0.9])
def test_extra_pairs_of_workers_without_data(P, mu):
    """Workers that never step need no data; an extra pair may average them all the same."""
    print("chains, perceptron, extra pairs of workers without data mu=%g" % mu, flush=True)
    n, dims, M, rows, K, T, stepping = 9, (40, 64, 5), 16, 48, 80, 2, 5
    d = dims[0] * dims[1] + dims[1] + dims[1] * dims[2] + dims[2]
    g = random_regular4_graph(n, 4)
    rng = np.random.default_rng(8)
    worker = rng.integers(0, stepping, K).astype(np.int32)
    sched = {"worker": worker, "neighbour": np.array([rng.choice(g[1][g[0][i]:g[0][i + 1]]) for i in worker], np.int32),
             "tau": np.minimum(rng.integers(0, T + 1, K), np.arange(K)).astype(np.int32),
             "batch_idx": rng.integers(0, rows, (K, M)).astype(np.int32)}
    extra = random_extra_pairs(g, sched["worker"], sched["neighbour"], max_extra=2, seed=2)
    assert (extra[1] >= stepping).any() and (extra[1] < stepping).any()
    feats, labels, _ = mixture_data(n, rows, din=dims[0], classes=dims[2], seed=9)
    x0 = np.stack([mlp_init(*dims, seed=s) for s in range(n)])
    eng = P.Engine(g, d, "mlp", M=M, gamma=0.05, T_max=T, mlp=dims, momentum=mu, weight_decay=1e-3 if mu else 0.0, verify_plan=True)
    eng.load_data(feats[:stepping], labels[:stepping])
    eng.set_models(x0, broadcast=False)
    eng.run_events(dict(sched, extra_pairs=extra))
    Xr, Vr = x0.copy(), np.zeros_like(x0)
    oracle.run_events(Xr, sched, oracle.MODEL_MLP, 0.05, M=M, gscale=1.0 / M, mlp=dims, features=feats, targets=labels, extra_pairs=extra,
                      momentum=mu, weight_decay=1e-3 if mu else 0.0, V=Vr if mu else None)
    # a hidden error next to a boundary of its bf16 rounding may fall on the other side: 2^-8 of one sample's share (1/16, times
    # an error of 0.1 and an input of 3) of a step of 0.05, 4e-6 an event and ten times that with momentum; 80 events
    assert np.max(np.abs(eng.get_models() - Xr)) <= 80 * (4e-5 if mu else 4e-6)
    eng.close()


def test_perceptron_with_more_inputs_than_a_grid_has_rows(P):
    """Update kernel: 32 inputs (16 with dense gradients) to a row of blocks, 65 535 rows to a launch."""
    import torch
    n, dims, gamma = 2, (2_097_160, 64, 2), 1.0
    d = dims[0] * dims[1] + dims[1] + dims[1] * dims[2] + dims[2]
    g = ring_graph(n)
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(5)
    scale = torch.full((d,), 0.3, device="cuda:0")
    scale[:dims[0] * dims[1]] = dims[0] ** -0.5
    x0 = torch.randn((n, d), device="cuda:0", generator=gen) * scale
    feats = [torch.randn((1, dims[0]), device="cuda:0", generator=gen).to(torch.bfloat16) for _ in range(n)]
    labels = [torch.zeros(1, dtype=torch.int32, device="cuda:0") for _ in range(n)]
    got = []
    for dense in (False, True):
        print("chains, perceptron with %d inputs, dense=%d" % (dims[0], dense), flush=True)
        eng = P.Engine(g, d, "mlp", M=1, gamma=gamma, T_max=0, mlp=dims, dense_gradient=dense, n_slots=1)
        eng.load_data(feats, labels)
        eng.h.set_models(x0.data_ptr(), d, on_device=True)
        eng.run_events({"worker": np.array([0], np.int32), "neighbour": np.array([1], np.int32), "tau": np.zeros(1, np.int32),
                        "batch_idx": np.zeros((1, 1), np.int32)})
        eng.h.synchronize()
        got.append((eng.X[:, :d].clone(), eng.Xbf16[:, :d].clone()))
        eng.close()
        del eng
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])
    assert torch.equal(got[0][1], got[0][0].to(torch.bfloat16))
    avg = (x0[0] + x0[1]) * 0.5
    assert torch.equal(got[0][0][1], avg)
    step = avg - got[0][0][0]
    inputs, hidden = dims[0], dims[1]
    error = step[inputs * hidden:inputs * hidden + hidden]                       # one sample: the gradient of b1 is dH itself
    assert int((error != 0).sum()) > hidden // 8
    want = feats[0][0].float()[:, None] * error[None, :]
    # the product of two bf16 values is exact; the step is what a subtraction from avg leaves: half a unit of the larger of them
    assert torch.all((step[:inputs * hidden].view(inputs, hidden) - want).abs() <= 2.0 ** -23 * torch.maximum(want.abs(), avg[:inputs * hidden].view(inputs, hidden).abs()) + 2.0 ** -23 * feats[0][0].float().abs()[:, None])
