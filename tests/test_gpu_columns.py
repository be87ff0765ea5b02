"""GPU: the synthetic model's events executed in one launch with strips of columns in LDS, against the same events
executed round by round (the caller's gradient function writes the generator's gradient): the same bits."""
import numpy as np
import pytest

import oracle
from workloads import random_extra_pairs, random_regular4_graph, ring_graph, with_identity_events

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1710_06952_amd as pkg
    pkg.lib()
    return pkg


# d around the float4, the strip widths of 4 ... 64 float4 columns and the blocks of four wavefronts; n up to the
# largest number of touched rows that the strips take (320, with momentum 160) and one more; then calls of few events per
# row, which go by rounds
@pytest.mark.parametrize("n,d,K,mu", [(5, 1, 40, 0.0), (5, 17, 40, 0.9), (6, 255, 60, 0.0), (6, 257, 60, 0.9), (9, 1023, 120, 0.0),
                                      (16, 4097, 200, 0.9), (64, 1030, 300, 0.0), (128, 515, 700, 0.0), (128, 515, 700, 0.9),
                                      (160, 70, 900, 0.9), (161, 70, 900, 0.9), (320, 66, 1500, 0.0), (321, 66, 1500, 0.0),
                                      (400, 130, 20, 0.0), (40, 100_003, 3, 0.9), (160, 500_001, 19, 0.0)])
def test_events_in_columns_are_the_events_of_the_rounds(P, n, d, K, mu):
    print("columns n=%d d=%d K=%d mu=%g" % (n, d, K, mu), flush=True)
    g = ring_graph(n) if n % 2 else random_regular4_graph(n, 3)
    T, std, seed, base = 4, float(np.float32(0.05)), (7 << 40) + 11, (3 << 33) + 5
    sched = oracle.make_schedule(g, K, seed=6, T_max=T)
    sched["neighbour"] = with_identity_events(sched["worker"], sched["neighbour"], 0.1, seed=1)
    sched["extra_pairs"] = random_extra_pairs(g, sched["worker"], sched["neighbour"], max_extra=1, seed=2)
    sched["gamma"] = (0.1 * (1 + np.arange(K) % 3)).astype(np.float32)
    x0 = np.random.default_rng(3).standard_normal((n, d)).astype(np.float32)
    kw = dict(gamma=0.1, T_max=T, momentum=mu, weight_decay=1e-3 if mu else 0.0)
    eng = P.Engine(g, d, "synth", synth_std=std, synth_seed=seed, **kw)
    ref = P.Engine(g, d, "external", **kw)

    def generator_gradient(requests, stream):
        for worker, event, xhat_ptr, g_ptr in requests:
            P.adpsgd_synth_gradient(seed, base + event, std, d, g_ptr, stream)

    for e in (eng, ref):
        e.set_models(x0, broadcast=False)
        e.h.set_event_count(base)
    eng.run_events(sched)
    ref.h.run_events_with(sched, generator_gradient)
    assert np.array_equal(eng.get_models(), ref.get_models())
    if mu:
        assert np.array_equal(eng.get_momentum(), ref.get_momentum())
    assert not eng.X[:, d:].any()                   # the padding of the rows stays zero
    st = eng.get_stats()
    touched = len(set(sched["worker"]) | set(sched["neighbour"]) | set(sched["extra_pairs"][1]) | set(sched["extra_pairs"][2]))
    assert st["events"] == K and 1 <= st["max_round_pairs"] <= n
    assert st["fused_launches"] == (1 if touched <= (160 if mu else 320) and K >= 2 * n else st["rounds"])
    assert ref.get_stats()["fused_launches"] == ref.get_stats()["rounds"]
    eng.close()
    ref.close()


# calls without extra pairs (a variant of its own), whose number of batches is odd and even: every event of a pair of workers
# depends on the one before, so K events are K batches; d with and without a tail
@pytest.mark.parametrize("d", [4096, 4099])
@pytest.mark.parametrize("K", [11, 12, 13])
@pytest.mark.parametrize("mu", [0.0, 0.9])
def test_calls_without_extra_pairs(P, K, d, mu):
    print("columns without extra pairs d=%d K=%d mu=%g" % (d, K, mu), flush=True)
    g, n = ring_graph(6), 6
    sched = oracle.make_schedule(g, K, seed=8, T_max=2)
    sched["worker"][:], sched["neighbour"][:] = 2, 3
    x0 = np.random.default_rng(5).standard_normal((n, d)).astype(np.float32)
    got = []
    for rounds in (False, True):
        eng = P.Engine(g, d, "synth", gamma=0.1, T_max=2, synth_std=0.3, synth_seed=5, momentum=mu, weight_decay=1e-3 if mu else 0.0,
                       verify_plan=True, rounds=rounds)
        eng.set_models(x0, broadcast=False)
        eng.run_events(sched)
        got.append((eng.get_models(), eng.get_momentum() if mu else None, eng.get_stats()["fused_launches"]))
        eng.close()
    assert (got[0][2], got[1][2]) == (1, K)
    assert np.array_equal(got[0][0], got[1][0])
    if mu:
        assert np.array_equal(got[0][1], got[1][1])


# a standard deviation that is a power of two has kernels of its own: each strip width, with and without momentum and extra pairs
@pytest.mark.parametrize("extra", [False, True])
@pytest.mark.parametrize("n,d,K,mu", [(5, 17, 40, 0.9), (6, 257, 60, 0.0), (64, 1030, 300, 0.0), (128, 515, 700, 0.9), (160, 70, 900, 0.9),
                                      (320, 66, 1500, 0.0), (6, 262_923, 60, 0.0), (13, 9109, 300, 0.9), (16, 2_000_001, 64, 0.0)])
def test_columns_with_a_power_of_two(P, n, d, K, mu, extra):
    print("columns n=%d d=%d K=%d mu=%g extra=%d" % (n, d, K, mu, extra), flush=True)
    g = ring_graph(n) if n % 2 else random_regular4_graph(n, 3)
    sched = oracle.make_schedule(g, K, seed=6, T_max=4)
    if extra:
        sched["extra_pairs"] = random_extra_pairs(g, sched["worker"], sched["neighbour"], max_extra=1, seed=2)
    x0 = np.random.default_rng(3).standard_normal((n, d)).astype(np.float32)
    out = []
    for rounds in (False, True):
        eng = P.Engine(g, d, "synth", gamma=0.1, T_max=4, synth_std=0.5, synth_seed=11, momentum=mu, weight_decay=1e-3 if mu else 0.0,
                       rounds=rounds)
        eng.set_models(x0, broadcast=False)
        eng.run_events(sched)
        out.append((eng.get_models(), eng.get_momentum() if mu else None, eng.get_stats()["fused_launches"]))
        eng.close()
    assert out[0][2] == 1 < out[1][2]
    assert np.array_equal(out[0][0], out[1][0])
    if mu:
        assert np.array_equal(out[0][1], out[1][1])
