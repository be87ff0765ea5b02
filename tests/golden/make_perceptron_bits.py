"""Records the results of short perceptron runs bit for bit: models, bf16 shadow, momentum buffers and losses.

tests/golden/perceptron_bits.npz was written by this script on an MI355X by the library as of commit 1d7ec0b, whose
second-layer gradients were formed on the vector ALUs as chains of fused multiply-adds (outputs in order; samples in
groups of four, the groups added as a pairwise tree).  Whatever forms these sums later has to keep that order.

    python tests/golden/make_perceptron_bits.py OUT.npz
"""
import os
import sys

import numpy as np

ROOT = os.path.dirname(os.path.dirname(os.path.dirname(os.path.abspath(__file__))))

# in, hidden, out, M, workers, momentum, wait-free
CASES = [(8, 64, 2, 1, 3, 0.0, False), (16, 64, 16, 64, 3, 0.0, False), (8, 128, 10, 33, 4, 0.9, False),
         (24, 192, 5, 47, 4, 0.9, True), (8, 1088, 4, 16, 2, 0.0, False), (40, 64, 7, 13, 5, 0.0, True)]


def results(P, case):
    """The arrays of one short run (staleness up to 3, 60 events)."""
    if ROOT not in sys.path:
        sys.path.insert(0, ROOT)
    import oracle
    from workloads import mixture_data, mlp_init, ring_graph
    din, hid, out, M, n, mu, comp = case
    d = din * hid + hid + hid * out + out
    g = ring_graph(n)
    feats, labels, _ = mixture_data(n, 64, din=din, classes=out, seed=12)
    sched = oracle.make_schedule(g, 60, seed=13, T_max=3, M=M, rows=[64] * n)
    eng = P.Engine(g, d, "mlp", M=M, gamma=0.02 if mu else 0.2, T_max=3, mlp=(din, hid, out), momentum=mu, weight_decay=1e-3 if mu else 0.0,
                   local_compensation=comp)
    eng.load_data(feats, labels)
    eng.set_models(mlp_init(din, hid, out, seed=14))
    eng.run_events(sched, want_loss=True)
    arrays = {"X": eng.get_models(), "b16": eng.get_bf16_models(), "loss": eng.get_loss()}
    if mu:
        arrays["V"] = eng.get_momentum()
    eng.close()
    return arrays


def name(case):
    return "_".join(str(int(10 * v) if isinstance(v, float) else int(v)) for v in case)


if __name__ == "__main__":
    sys.path.insert(0, os.getcwd())          # the tree whose library is recorded
    import paper_1710_06952_amd as P
    rec = {}
    for case in CASES:
        print(name(case), flush=True)
        for k, v in results(P, case).items():
            rec[name(case) + "/" + k] = v
    np.savez_compressed(sys.argv[1], **rec)
