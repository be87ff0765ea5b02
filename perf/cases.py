"""What a user of this library has it do, as cases that can be timed and compared.

A case names a call and its sizes; ``prepare`` makes what a program holds before that call (an engine with
its data, models and schedule in place), ``run`` is one call through the public entry points, ``exact`` the
same result in 64-bit arithmetic from plain torch.

kinds  events    Engine.run_events on a seeded schedule (models synth, lsq, logreg, mlp)
       external  Engine.run_events_with: the gradient is a function of the caller
       sync      Engine.run_sync_steps, the synchronous comparison schedule
       diagnose  mean model, consensus distance, divergence check and, with data, objective and error
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_1710_06952_amd as P
from workloads import (hop_ring_graph, linear_data_on_device, mixture_data_on_device, mlp_init,
                       random_regular4_graph, ring_graph)

DEVICE = "cuda:0"

_DEFAULTS = dict(kind="events", graph="ring", M=0, rows=0, K=0, T_max=0, momentum=0.0, weight_decay=0.0,
                 wait_free=False, loss=False, slow=0, mlp_in=0, mlp_hidden=0, mlp_out=0)


def _case(**kw):
    c = dict(_DEFAULTS)
    c.update(kw)
    if c["model"] == "mlp":
        c["d"] = c["mlp_in"] * c["mlp_hidden"] + c["mlp_hidden"] + c["mlp_hidden"] * c["mlp_out"] + c["mlp_out"]
    return c


def listed():
    return [
        # the benchmark's headline shape: 128 replicas of 25.6 M parameters on a ring, gradients drawn by the library
        _case(name="gossip", model="synth", n=128, d=25_600_000, K=2000, T_max=16),
        # the same workload with the experiments' optimizer on a random 4-regular graph, odd number of parameters
        _case(name="gossip_momentum", model="synth", graph="reg4", n=32, d=3_000_001, K=500, T_max=16, momentum=0.9, weight_decay=1e-4),
        # the smallest training call: least squares, 1024 parameters, a tenth of the configuration's events
        _case(name="lsq_short", model="lsq", n=8, d=1024, M=32, rows=1024, K=200, T_max=3),
        # the slow-worker study's shape: 16 workers, 4096 parameters, small minibatches, losses recorded
        _case(name="lsq_study", model="lsq", n=16, d=4096, M=8, rows=1024, K=1280, T_max=24, loss=True),
        # logistic regression on dense features, the minibatch rows are the traffic
        _case(name="logreg", model="logreg", n=64, d=65536, M=128, rows=1024, K=500, T_max=8, loss=True),
        # wait-free variant with the experiments' optimizer (what the paper's runs used), ragged sizes
        _case(name="waitfree", model="logreg", graph="reg4", n=16, d=20_001, M=50, rows=700, K=400, T_max=6, momentum=0.9,
              weight_decay=1e-4, wait_free=True),
        # a long model: least squares with 4 M parameters, four slow workers, long staleness
        _case(name="lsq_long", model="lsq", graph="reg4", n=32, d=4 * 1024 * 1024, M=8, rows=16, K=200, T_max=128, slow=4),
        # the perceptron, 784-1024-10, bf16 inputs and shadow weights
        _case(name="mlp", model="mlp", graph="reg4", n=16, mlp_in=784, mlp_hidden=1024, mlp_out=10, M=64, rows=2048, K=1000, T_max=4),
        # the convergence study's network and optimizer, an epoch per call, losses recorded
        _case(name="mlp_momentum", model="mlp", n=16, mlp_in=64, mlp_hidden=256, mlp_out=10, M=32, rows=2048, K=1024, T_max=4,
              momentum=0.9, weight_decay=1e-4, loss=True),
        # gradients from the caller (a torch function), with momentum: the library averages and applies
        _case(name="external", kind="external", model="external", n=8, d=12_000_003, K=60, T_max=4, momentum=0.9, weight_decay=1e-4),
        # the synchronous comparison schedule on the same kind of data, odd number of parameters
        _case(name="sync", kind="sync", model="lsq", n=32, d=1_000_003, M=8, rows=16, K=10),
        # what a run reports between calls: mean model, consensus distance, divergence check at a large shape
        _case(name="diagnose", kind="diagnose", model="synth", n=64, d=25_600_000),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the ranges the listed ones stand for."""
    kind = rng.choice(["synth", "synth", "lsq", "lsq", "logreg", "mlp", "external", "sync", "diagnose"])
    n = _log_int(rng, 5, 64)
    graph = rng.choice(["ring", "reg4", "hop"])
    optim = dict(momentum=0.9, weight_decay=1e-4) if rng.random() < 0.4 else {}
    T = rng.choice([0, 3, 8, 16, 40])
    if kind == "synth":
        n = _log_int(rng, 5, 128)
        d = _log_int(rng, 5_000, 25_600_000)
        return _case(model="synth", graph=graph, n=n, d=d, K=_log_int(rng, 50, 2000), T_max=T, **optim)
    if kind in ("lsq", "logreg"):
        M = _log_int(rng, 1, 128)
        d = _log_int(rng, 300, min(4_200_000, 33_600_000 // M))
        rows = max(M, min(2048, 1_000_000_000 // (n * d)))
        K = max(20, min(_log_int(rng, 50, 1500), 30_000_000_000 // (M * d)))
        return _case(model=kind, graph=graph, n=n, d=d, M=M, rows=rows, K=K, T_max=T, loss=rng.random() < 0.5,
                     wait_free=rng.random() < 0.3, **optim)
    if kind == "mlp":
        return _case(model="mlp", graph=graph, n=min(n, 32), mlp_in=8 * rng.randint(4, 128), mlp_hidden=64 * rng.randint(1, 16),
                     mlp_out=rng.randint(2, 16), M=rng.randint(1, 64), rows=rng.choice([256, 1000, 2048]), K=_log_int(rng, 50, 1000),
                     T_max=T, loss=rng.random() < 0.5, wait_free=rng.random() < 0.3, **optim)
    if kind == "external":
        return _case(kind="external", model="external", graph=graph, n=min(n, 16), d=_log_int(rng, 10_000, 12_000_000),
                     K=_log_int(rng, 20, 100), T_max=min(T, 16), **optim)
    if kind == "sync":
        model = rng.choice(["synth", "lsq", "mlp"])
        if model == "synth":
            return _case(kind="sync", model="synth", graph=graph, n=n, d=_log_int(rng, 20_000, 12_000_000), K=rng.randint(2, 20), **optim)
        if model == "mlp":
            return _case(kind="sync", model="mlp", graph=graph, n=min(n, 16), mlp_in=8 * rng.randint(4, 64),
                         mlp_hidden=64 * rng.randint(1, 8), mlp_out=10, M=32, rows=512, K=rng.randint(2, 40), **optim)
        d = _log_int(rng, 1_000, 1_000_000)
        return _case(kind="sync", model="lsq", graph=graph, n=n, d=d, M=8, rows=16, K=rng.randint(2, 20), **optim)
    if rng.random() < 0.5:
        return _case(kind="diagnose", model="synth", graph=graph, n=n, d=_log_int(rng, 50_000, 25_600_000))
    if rng.random() < 0.5:
        return _case(kind="diagnose", model="mlp", graph=graph, n=min(n, 16), mlp_in=8 * rng.randint(4, 100),
                     mlp_hidden=64 * rng.randint(1, 16), mlp_out=10, M=64, rows=rng.choice([1000, 2048]))
    d = _log_int(rng, 1_000, 500_000)
    return _case(kind="diagnose", model="logreg", graph=graph, n=n, d=d, M=8, rows=max(8, min(2048, 1_000_000_000 // (n * d))))


# ---- what the program holds before the call ---------------------------------------------------------------------

SYNTH_STD = float(np.float32(0.0316227766016838))      # variance 1e-3
LAMBDA = 1e-4


def _graph(case):
    return {"ring": ring_graph, "reg4": lambda n: random_regular4_graph(n, 0), "hop": hop_ring_graph}[case["graph"]](case["n"])


def _gamma(case):
    """Step sizes at which the runs are stable however long they go on."""
    gamma = {"synth": 0.1, "external": 0.2, "lsq": 0.5 * case["M"], "logreg": 0.5 * case["M"], "mlp": 0.05}[case["model"]]
    if case["kind"] == "events" and case["T_max"] > 4:
        gamma *= 0.5
    return gamma * (0.1 if case["momentum"] else 1.0)


def _mlp(case):
    return (case["mlp_in"], case["mlp_hidden"], case["mlp_out"])


def _data(case, seed):
    n, rows = case["n"], case["rows"]
    if case["model"] == "mlp":
        return mixture_data_on_device(n, rows, din=case["mlp_in"], classes=case["mlp_out"], seed=seed, device=DEVICE)
    features, labels = linear_data_on_device(case["model"], n, rows, case["d"], seed=seed, device=DEVICE)
    extra = -case["d"] % 4                     # the library takes rows whose length is a multiple of 4
    return [torch.nn.functional.pad(f, (0, extra)) if extra else f for f in features], labels


def _x0(case, seed):
    """The equal initial model (one vector), and per-worker deviations for the diagnostics."""
    if case["model"] == "mlp":
        return torch.from_numpy(mlp_init(*_mlp(case), seed=seed)).to(DEVICE)
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(7919 * seed + 5)
    scale = 1.0 if case["model"] == "external" else 0.1
    return torch.randn(case["d"], device=DEVICE, generator=gen) * scale


def _spread(case, seed):
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(7919 * seed + 6)
    return torch.randn((case["n"], case["d"]), device=DEVICE, generator=gen) * 0.01


def _targets(case, seed):
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(7919 * seed + 7)
    return torch.randn((case["n"], case["d"]), device=DEVICE, generator=gen)


def _schedule(case, graph, seed):
    n = case["n"]
    kw = dict(seed=seed, T_max=case["T_max"], M=case["M"], rows=[max(case["rows"], 1)] * n)
    if case["slow"]:
        slow = np.arange(n) < case["slow"]
        kw.update(tau_mode=1, weight=np.where(slow, 1, 10), tau_num=np.where(slow, 20, 2), tau_den=np.where(slow, 21, 3))
    return P.adpsgd_make_schedule(graph, case["K"], **kw)


def _sync_batch(case, seed):
    if case["M"] == 0:
        return None
    rng = np.random.default_rng([seed, 31])
    return rng.integers(0, case["rows"], size=(case["K"], case["n"], case["M"])).astype(np.int32)


def _prob(case):
    p = np.arange(1, case["n"] + 1, dtype=np.float64)
    return p / p.sum()


def prepare(case, seed):
    graph = _graph(case)
    kind, model, n = case["kind"], case["model"], case["n"]
    slots = dict(n_slots=max(n, case["T_max"] + 1)) if kind == "sync" else {}
    eng = P.Engine(graph, case["d"], model, M=case["M"], gamma=_gamma(case), lam=LAMBDA if model == "logreg" else 0.0,
                   T_max=case["T_max"], synth_std=SYNTH_STD, synth_seed=seed, mlp=_mlp(case), momentum=case["momentum"],
                   weight_decay=case["weight_decay"], local_compensation=case["wait_free"], device=DEVICE, **slots)
    if model in ("lsq", "logreg", "mlp"):
        eng.load_data(*_data(case, seed))
    x0 = _x0(case, seed)
    if kind == "diagnose":
        x = x0 + _spread(case, seed)
        eng.h.set_models(x.data_ptr(), case["d"], on_device=True)
        return {"case": case, "eng": eng, "p": _prob(case), "mean": torch.empty(case["d"], dtype=torch.float32, device=DEVICE)}
    eng.h.set_models(x0.data_ptr(), 0, on_device=True)
    state = {"case": case, "eng": eng}
    if kind == "sync":
        state["batch"] = _sync_batch(case, seed)
    else:
        state["schedule"] = _schedule(case, graph, seed)
    if kind == "external":
        targets = _targets(case, seed)

        def gradient(worker, event, xhat, g):      # F_i(x) = |x - t_i|^2 / 2
            torch.sub(xhat, targets[worker], out=g)

        state["gradient"] = gradient
    torch.cuda.synchronize()
    return state


def run(state):
    case, eng = state["case"], state["eng"]
    kind = case["kind"]
    if kind == "diagnose":
        eng.h.mean_model_to_device(state["mean"].data_ptr())
        out = {"mean": state["mean"], "consensus": eng.consensus_distance(), "consensus_p": eng.consensus_distance(state["p"]),
               "nonfinite": eng.count_nonfinite()}
        if case["model"] != "synth":
            out["objective"] = eng.objective()
            out["error"] = eng.classification_error()
        return out
    if kind == "sync":
        eng.run_sync_steps(case["K"], state["batch"], want_loss=case["loss"])
    elif kind == "external":
        eng.run_events_with(state["schedule"], state["gradient"])
    else:
        eng.run_events(state["schedule"], want_loss=case["loss"])
    out = {"X": eng.X}
    if eng.V is not None:
        out["V"] = eng.V
    if eng.Xbf16 is not None:
        out["Xbf16"] = eng.Xbf16
    if case["loss"]:
        out["loss"] = eng.loss
    return out


# ---- what a call cannot do without --------------------------------------------------------------------------------

def work(case):
    """Models (and momentum buffers, bf16 shadows) read and written once per call, the minibatch rows that the call
    names read once, plus what the caller's gradient function sees and writes for every event; the arithmetic of
    the gradients and updates (a normal variate counted as 60 operations)."""
    n, d, M, K, model = case["n"], case["d"], case["M"], case["K"], case["model"]
    row = 2 * case["mlp_in"] if model == "mlp" else 4 * d
    if case["kind"] == "diagnose":
        nbytes, flops = 4.0 * n * d + 4.0 * d, 8.0 * n * d
        if model != "synth":
            nbytes += float(n) * case["rows"] * row
            flops += 2.0 * n * case["rows"] * (case["mlp_hidden"] * (case["mlp_in"] + case["mlp_out"]) if model == "mlp" else d)
        return {"bytes": nbytes, "flops": flops}
    updates = K * n if case["kind"] == "sync" else K
    optim = bool(case["momentum"])
    touched = n if case["kind"] == "sync" else min(n, 2 * K)
    nbytes = 8.0 * touched * d * (2 if optim else 1) + (4.0 * touched * d if model == "mlp" else 0.0)
    flops = updates * d * (8.0 if optim else 4.0)
    if model == "synth":
        flops += 60.0 * updates * d
    elif model == "external":
        nbytes = updates * d * 4.0 * (4 + 4 + (2 if optim else 0))     # x^, target, g out and in; both rows in and out; v
        flops += updates * d
    else:
        nbytes += float(min(updates * M, n * case["rows"])) * row
        if model == "mlp":
            flops += updates * M * (4.0 * case["mlp_in"] * case["mlp_hidden"] + 6.0 * case["mlp_hidden"] * case["mlp_out"])
        else:
            flops += 4.0 * updates * M * d
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """About four times the error against ``exact`` measured at the listed and at drawn sizes: 5e-8 ... 5e-7 for the
    32-bit models; for the perceptron 1e-6 ... 5e-6 on the weights, 5e-5 ... 9e-5 on their bf16 shadow (a weight near a
    rounding boundary) and 2e-4 ... 5e-4 on the momentum buffers (an activation near one)."""
    if case["model"] == "mlp" and case["kind"] != "diagnose":
        return {"rel": 2e-3 if case["momentum"] else 4e-4}
    return {"rel": 2e-6}


# ---- the same in 64 bits ---------------------------------------------------------------------------------------------

def _hi_lo(a, b):
    """High and low word of the product of 32-bit words held in int64 (the wrapped product has the right bits)."""
    prod = a * b
    return (prod >> 32) & 0xFFFFFFFF, prod & 0xFFFFFFFF


def _normals(seed, k, d):
    """g_k / std of the library's counter-based generator: Philox4x32-10 and Box-Muller."""
    q = torch.arange((d + 3) // 4, dtype=torch.int64, device=DEVICE)
    c0, c1 = q & 0xFFFFFFFF, q >> 32
    c2 = torch.full_like(q, k & 0xFFFFFFFF)
    c3 = torch.full_like(q, ((k >> 32) & 0x00FFFFFF) | (2 << 24))
    k0, k1 = seed & 0xFFFFFFFF, (seed >> 32) & 0xFFFFFFFF
    for _ in range(10):
        h0, l0 = _hi_lo(c0, 0xD2511F53)
        h1, l1 = _hi_lo(c2, 0xCD9E8D57)
        c0, c1, c2, c3 = h1 ^ c1 ^ k0, l1, h0 ^ c3 ^ k1, l0
        k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
    out = torch.empty((q.numel(), 4), dtype=torch.float64, device=DEVICE)
    for t, (a, b) in enumerate(((c0, c1), (c2, c3))):
        r = torch.sqrt(-2.0 * torch.log(((a >> 9).double() + 0.5) * 2.0 ** -23))
        angle = 2.0 * math.pi * (b >> 8).double() * 2.0 ** -24
        out[:, 2 * t] = r * torch.cos(angle)
        out[:, 2 * t + 1] = r * torch.sin(angle)
    return out.reshape(-1)[:d]


def _bf16(x):
    return x.to(torch.bfloat16).double()


class _Gradients:
    """Minibatch gradient and loss of worker i at xhat (float64), by model."""

    def __init__(self, case, seed):
        self.case, self.seed = case, seed
        if case["model"] in ("lsq", "logreg", "mlp"):
            self.features, self.labels = _data(case, seed)
        if case["model"] == "external":
            self.targets = _targets(case, seed)

    def __call__(self, i, event, xhat, idx):
        case = self.case
        model, M = case["model"], case["M"]
        if model == "synth":
            return _normals(self.seed, event, case["d"]) * SYNTH_STD, None
        if model == "external":
            return xhat - self.targets[i].double(), None
        idx = torch.from_numpy(idx.astype(np.int64)).to(DEVICE)
        if model == "mlp":
            return self._mlp(i, xhat, idx)
        A, t = self.features[i][idx][:, :case["d"]].double(), self.labels[i][idx].double()
        z = A @ xhat
        if model == "lsq":
            return A.t() @ (z - t) / M, 0.5 * ((z - t) ** 2).mean()
        s = -t * z
        loss = torch.nn.functional.softplus(s).mean() + 0.5 * LAMBDA * xhat.dot(xhat)
        return A.t() @ (-t * torch.sigmoid(s)) / M + LAMBDA * xhat, loss

    def _mlp(self, i, xhat, idx):      # the path's own 16-bit roundings: shadow weights, activations, their error
        din, hid, out = _mlp(self.case)
        M = self.case["M"]
        w = _bf16(xhat)
        W1, b1 = w[:din * hid].view(din, hid), w[din * hid:din * hid + hid]
        W2, b2 = w[din * hid + hid:din * hid + hid + hid * out].view(hid, out), w[-out:]
        x, y = self.features[i][idx][:, :din].double(), self.labels[i][idx].long()
        H = _bf16(torch.relu(x @ W1 + b1))
        logits = H @ W2 + b2
        dl = torch.softmax(logits, 1)
        loss = torch.nn.functional.cross_entropy(logits, y)
        dl[torch.arange(M, device=DEVICE), y] -= 1.0
        dH = torch.where(H > 0, _bf16((dl @ W2.t()) / M), torch.zeros_like(H))
        g = torch.cat([(x.t() @ dH).reshape(-1), dH.sum(0), (H.t() @ dl / M).reshape(-1), dl.sum(0) / M])
        return g, loss


def _pad(x, ld):
    out = torch.zeros((x.shape[0], ld), dtype=torch.float64, device=DEVICE)
    out[:, :x.shape[1]] = x
    return out


def exact(case, seed):
    kind, model, n, d = case["kind"], case["model"], case["n"], case["d"]
    if kind == "diagnose":
        return _exact_diagnose(case, seed)
    updates = case["K"] * (n if kind == "sync" else 1)
    per = 6e-10 * d if model == "synth" else 1.2e-11 * (3 * case["M"] * d + 40 * d)
    if updates * (per + 6e-4) > 15.0:
        return None
    grads = _Gradients(case, seed)
    gamma = float(np.float32(_gamma(case)))
    mu, wd = float(np.float32(case["momentum"])), float(np.float32(case["weight_decay"]))
    X = _x0(case, seed).double().repeat(n, 1)
    V = torch.zeros_like(X) if mu else None
    loss = torch.zeros(updates, dtype=torch.float64, device=DEVICE)

    def step(i, avg, g):
        if not mu:
            return avg - gamma * g
        V[i] = mu * V[i] + (g + wd * avg)
        return avg - gamma * V[i]

    if kind == "sync":
        rowptr, col = _graph(case)
        degree = np.diff(rowptr)
        batch = _sync_batch(case, seed)
        for t in range(case["K"]):
            new = torch.empty_like(X)
            for i in range(n):
                g, value = grads(i, t * n + i, X[i], None if batch is None else batch[t, i])
                if value is not None:
                    loss[t * n + i] = value
                nb = col[rowptr[i]:rowptr[i + 1]]
                w = [1.0 / (1.0 + max(degree[i], degree[j])) for j in nb]      # Metropolis weights
                mixed = X[i] * float(np.float32(1.0 - sum(w)))
                for j, wj in zip(nb, w):
                    mixed = mixed + X[j] * float(np.float32(wj))
                new[i] = step(i, mixed, g)
            X = new
    else:
        s = _schedule(case, _graph(case), seed)
        worker, tau, batch = s["worker"], s["tau"], s["batch_idx"]
        due = [[] for _ in range(case["K"])]       # events whose stale read happens before event t
        previous, latest = {}, {}
        for k in range(case["K"]):
            t = k if model == "synth" else k - int(tau[k])
            due[t].append(k)
            previous[k] = latest.get(int(worker[k]))
            latest[int(worker[k])] = k
        pending = {}
        for t in range(case["K"]):
            for k in due[t]:
                xhat, kp = X[worker[k]], previous[k]
                if case["wait_free"] and kp is not None and kp - int(tau[kp]) <= t <= kp:
                    xhat = xhat - gamma * pending[kp]
                pending[k], value = grads(int(worker[k]), k, xhat, None if batch is None else batch[k])
                if value is not None:
                    loss[k] = value
            i, j = int(worker[t]), int(s["neighbour"][t])
            avg = (X[i] + X[j]) * 0.5
            X[j] = avg
            X[i] = step(i, avg, pending[t])
            del pending[t]
    ld = (d + 63) // 64 * 64
    out = {"X": _pad(X, ld)}
    if mu:
        out["V"] = _pad(V, ld)
    if model == "mlp":
        out["Xbf16"] = _pad(_bf16(X), ld)
    if case["loss"]:
        out["loss"] = loss
    return out


def _exact_diagnose(case, seed):
    n, d, p = case["n"], case["d"], torch.from_numpy(_prob(case)).to(DEVICE)
    X = _x0(case, seed) + _spread(case, seed)          # rounded to 32 bits as the models are
    mean = torch.zeros(d, dtype=torch.float64, device=DEVICE)
    for i in range(n):
        mean += X[i].double()
    mean /= n
    sq = torch.stack([((X[i].double() - mean) ** 2).sum() for i in range(n)])
    out = {"mean": mean, "consensus": float(sq.mean()), "consensus_p": float((sq * p).sum()), "nonfinite": 0}
    if case["model"] == "synth":
        return out
    features, labels = _data(case, seed)
    at = mean.float().double()
    f = err = 0.0
    for i in range(n):
        if case["model"] == "mlp":
            din, hid, o = _mlp(case)
            w = _bf16(at)
            H = _bf16(torch.relu(features[i][:, :din].double() @ w[:din * hid].view(din, hid) + w[din * hid:din * hid + hid]))
            logits = H @ w[din * hid + hid:din * hid + hid + hid * o].view(hid, o) + w[-o:]
            f += float(torch.nn.functional.cross_entropy(logits, labels[i].long())) / n
            err += float((logits.argmax(1) != labels[i]).double().mean()) / n
        else:
            z, t = features[i][:, :d].double() @ at, labels[i].double()
            f += float(torch.nn.functional.softplus(-t * z).mean() + 0.5 * LAMBDA * at.dot(at)) / n
            err += float((torch.where(z >= 0, 1.0, -1.0) != t).double().mean()) / n
    out["objective"] = f
    out["error"] = err
    return out
