"""GPU: chains of four updates of the perceptron (up to 2^18 parameters, no momentum) and of three (beyond), next to the line between
them: factored and dense gradients give the same bits, the models agree with the oracle's, and the longer chains take fewer rounds."""
import numpy as np
import pytest

import oracle
from workloads import mixture_data, mlp_init, random_regular4_graph

pytestmark = pytest.mark.gpu


LINE = 2 ** 18
DIMS = [(248, 1024, 6), (248, 1024, 7)]          # one at the line, one beyond


def _size(dims):
    return dims[0] * dims[1] + dims[1] + dims[1] * dims[2] + dims[2]


def test_next_to_the_line():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1710_06952_amd as P
    assert LINE - 1024 < _size(DIMS[0]) <= LINE < _size(DIMS[1]) < LINE + 1024
    n, rows, K, M, T = 12, 48, 60, 20, 5
    g = random_regular4_graph(n, 4)
    sched = oracle.make_schedule(g, K, seed=9, T_max=T, M=M, rows=[rows] * n)
    rounds = []
    for dims in DIMS:
        print("perceptron chains %s" % (dims,), flush=True)
        feats, labels, _ = mixture_data(n, rows, din=dims[0], classes=dims[2], seed=9)
        x0 = mlp_init(*dims, seed=9)
        out = []
        for dense in (False, True):
            eng = P.Engine(g, _size(dims), "mlp", M=M, gamma=0.02, T_max=T, mlp=dims, dense_gradient=dense, verify_plan=True)
            eng.load_data(feats, labels)
            eng.set_models(x0)
            eng.run_events(sched)
            out.append((eng.get_models(), eng.get_bf16_models()))
            rounds.append(eng.get_stats()["rounds"])
            eng.close()
        assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1])
        Xr = np.repeat(x0[None], n, axis=0).astype(np.float32)
        oracle.run_events(Xr, sched, oracle.MODEL_MLP, 0.02, M=M, gscale=1.0 / M, features=feats, targets=labels, mlp=dims)
        err = np.max(np.abs(out[0][0].astype(np.float64) - Xr)) / np.max(np.abs(Xr))
        assert err <= 2e-3, err          # bf16 activations next to a rounding boundary, as in the other tests of this model
    assert rounds[0] == rounds[1] < rounds[2] == rounds[3], rounds      # the same schedule, fewer rounds with the longer chains
