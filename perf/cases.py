"""Timed workloads of the framework, each through a public entry point.

A case is a dict of plain values. ``prepare`` makes what a user's program holds
before the call (bit rows, angles, a batch plan, a trainer) on the GPU from a
seed, ``run`` makes one pass, ``work`` counts what a pass cannot do without and
``exact`` evaluates the same inputs in FP64 with plain torch.

Kinds
  expval   forward only: means and standard errors of a given circuit
  grad     autograd forward + backward of the expectation values
  mmd      autograd forward + backward of the MMD^2 loss
  batch    forward + backward of many circuits of uneven size (BatchPlan)
  indep    forward + backward with a sample set per observable
  bitflip  forward + backward of the exact bitflip product form
  train    one training step on the device (Trainer)
"""
import math
import random

import numpy as np
import torch

from paper_2501_04776_amd import (BatchPlan, Circuit, IQPBitflipExpval, IQPExpval, IQPMMDLoss,
                                  Trainer, iqp_expval, iqp_expval_indep, iqp_expval_indep_grad)

DEV = "cuda"
SIGMAS = (1.0, 5.0, 17.0)
DENSE = ("split_bf16", "split3_bf16", "split_bf16_fp8", "fp32")


def listed():
    return [
        # the first thing a user runs: a 10-qubit circuit of all local gates
        {"name": "expval_n10", "kind": "expval", "n": 10, "local": True, "l": 100, "s": 1000,
         "op_w": 3, "theta": 3.14159, "prec": "split_bf16"},
        # a small optimisation step: forward and backward, launch-bound
        {"name": "grad_n70", "kind": "grad", "n": 70, "m": 700, "l": 150, "s": 600, "gate_w": 4,
         "op_w": 4, "theta": 3.14159, "prec": "split3_bf16"},
        # the 300-qubit, 45150-parameter circuit: one optimisation step
        {"name": "grad_n300", "kind": "grad", "n": 300, "local": True, "l": 1000, "s": 10000,
         "op_w": -2, "theta": -0.1, "prec": "split_bf16"},
        # the same circuit in the sparse form
        {"name": "grad_n300_sparse", "kind": "grad", "n": 300, "local": True, "l": 1000,
         "s": 10000, "op_w": -2, "theta": -0.1, "prec": "sparse_fp32"},
        # and in the FP32 form, at odd sizes
        {"name": "grad_n300_fp32", "kind": "grad", "n": 300, "local": True, "l": 517, "s": 2501,
         "op_w": -2, "theta": -0.1, "prec": "fp32"},
        # a 1000-qubit circuit of 100000 random gates, sparse form
        {"name": "grad_n1000_sparse", "kind": "grad", "n": 1000, "m": 100000, "l": 2000,
         "s": 10000, "gate_w": 3, "op_w": 10, "theta": 3.14159, "prec": "sparse_fp32"},
        # MMD loss and gradient with three kernel bandwidths
        {"name": "mmd_n300", "kind": "mmd", "n": 300, "local": True, "per_sigma": 2000,
         "s": 10000, "N": 2000, "theta": -0.1, "prec": "split_bf16_fp8"},
        # many circuits of uneven size in one pass
        {"name": "batch16", "kind": "batch", "count": 16, "shapes": 505, "n_max": 2000,
         "m_max": 200000, "l_max": 5000, "s": 4096, "gate_w": 4, "op_w": 4, "theta": 3.14159,
         "prec": "split_bf16"},
        # estimation only: many observables and samples of a small circuit
        {"name": "expval_n100_m1000", "kind": "expval", "n": 100, "m": 1000, "l": 10000,
         "s": 10000, "gate_w": 0, "op_w": 0, "theta": 3.14159, "prec": "split_bf16"},
        # uncorrelated estimates: every observable with its own samples
        {"name": "indep_n300", "kind": "indep", "n": 300, "local": True, "l": 300, "s": 10000,
         "op_w": -2, "theta": -0.1},
        # the exact bitflip form of a large circuit
        {"name": "bitflip_n1000", "kind": "bitflip", "n": 1000, "m": 100000, "l": 10000,
         "gate_w": 3, "op_w": 10, "theta": -0.1},
        # one training step: sampling, loss, gradient, Adam
        {"name": "train_n300", "kind": "train", "n": 300, "local": True, "per_sigma": 2000,
         "s": 10000, "N": 2000, "theta": -0.1, "prec": "split_bf16", "auto": True},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["expval", "expval", "grad", "grad", "grad", "mmd", "batch", "indep",
                       "bitflip", "train"])
    c = {"kind": kind, "theta": -0.1 if kind == "bitflip" else rng.choice([3.14159, -0.1])}
    if kind == "batch":
        c.update(count=rng.randint(4, 14), shapes=rng.randint(1, 10 ** 6),
                 n_max=_log(rng, 100, 2000), m_max=_log(rng, 2000, 150000),
                 l_max=_log(rng, 200, 4000), s=_log(rng, 500, 4096), gate_w=4, op_w=4,
                 prec=rng.choice(DENSE[:3]))
        return c
    c["n"] = _log(rng, 10, 1000)
    if kind in ("mmd", "train") or rng.random() < 0.3:
        c["n"] = min(c["n"], 300)
        c["local"] = True
        m = c["n"] * (c["n"] + 1) // 2
    else:
        m = c["m"] = _log(rng, 50, 100000)
        c["gate_w"] = rng.choice([0, 3, 4])
    c["s"] = _log(rng, 500, 10000)
    if kind in ("mmd", "train"):
        c["per_sigma"] = _log(rng, 50, 2000)
        c["N"] = _log(rng, 100, 2000)
        c["prec"] = rng.choice(DENSE[:3] + ("sparse_fp32",))
        if kind == "train":
            c["auto"] = rng.random() < 0.5
        return c
    c["op_w"] = rng.choice([0, 3, 4, -2])
    c["l"] = _log(rng, 50, 10000)
    if kind in ("expval", "grad"):
        c["prec"] = rng.choice(DENSE + ("sparse_fp32", "sparse_fp32"))
        top = 2e11 if c["prec"] == "fp32" else 2e12
        c["l"] = max(50, min(c["l"], int(top / (m * c["s"]))))
    elif kind == "indep":
        c["l"] = min(c["l"], 1000)
    return c


# --- inputs -------------------------------------------------------------------
def _pack(bits):
    """0/1 rows [count][n] -> packed int64 words [count][ceil(n / 64)]."""
    count, n = bits.shape
    W = (n + 63) // 64
    out = torch.zeros((count, W), dtype=torch.int64, device=bits.device)
    for q in range(min(n, 64)):
        cols = bits[:, q::64].to(torch.int64)
        out[:, :cols.shape[1]] |= cols << q
    return out


def _local(n):
    q = torch.triu_indices(n, n, 1, device=DEV)
    m = n + q.shape[1]
    bits = torch.zeros((m, n), dtype=torch.bool, device=DEV)
    bits[:n] = torch.eye(n, dtype=torch.bool, device=DEV)
    rows = torch.arange(n, m, device=DEV)
    bits[rows, q[0]] = True
    bits[rows, q[1]] = True
    return bits


def _rows(g, count, n, w):
    """Random strings: weight uniform in 1..w, exactly -w for w < 0, or
    Bernoulli(3/n) bits for w = 0."""
    if w == 0:
        return torch.rand((count, n), generator=g, device=DEV) < 3.0 / n
    top = min(abs(w), n)
    first = torch.randint(0, n, (count, 1), generator=g, device=DEV)
    # distinct qubits: steps of at least 1 that together stay below n
    span = max(1, (n - 1) // max(1, top - 1))
    step = torch.randint(1, span + 1, (count, top), generator=g, device=DEV)
    step[:, 0] = 0
    q = (first + torch.cumsum(step, 1)) % n
    if w < 0:
        keep = torch.ones((count, top), dtype=torch.bool, device=DEV)
    else:
        wt = torch.randint(1, top + 1, (count, 1), generator=g, device=DEV)
        keep = torch.arange(top, device=DEV)[None, :] < wt
    bits = torch.zeros((count, n), dtype=torch.int8, device=DEV)
    bits.scatter_add_(1, q, keep.to(torch.int8))
    return bits > 0


def _angles(g, m, scale):
    """theta ~ U(-scale, scale), or N(0, scale^2) for a negative scale."""
    if scale < 0:
        return torch.randn(m, generator=g, device=DEV, dtype=torch.float64) * -scale
    return (torch.rand(m, generator=g, device=DEV, dtype=torch.float64) * 2 - 1) * scale


def _uniform(g, shape, n):
    W = (n + 63) // 64
    words = torch.randint(-2 ** 63, 2 ** 63 - 1, tuple(shape) + (W,), generator=g, device=DEV,
                          dtype=torch.int64)
    if n % 64:
        words[..., -1] &= (1 << (n % 64)) - 1
    return words


def _sigma_prob(sigma):
    return (1.0 - math.exp(-1.0 / (2.0 * sigma * sigma))) / 2.0


def _gates(g, case, n, m):
    return _local(n) if case.get("local") else _rows(g, m, n, case["gate_w"])


def _gate_count(case):
    n = case["n"]
    return n * (n + 1) // 2 if case.get("local") else case["m"]


def _shapes(case):
    r = random.Random(case["shapes"])
    return [(r.randint(min(50, case["n_max"]), case["n_max"]),
             r.randint(min(1000, case["m_max"]), case["m_max"]),
             r.randint(min(100, case["l_max"]), case["l_max"])) for _ in range(case["count"])]


def _inputs(case, seed):
    """The raw inputs of a case (bit rows as 0/1 and packed, angles, ...)."""
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    kind = case["kind"]
    if kind == "batch":
        out = []
        for n, m, l in _shapes(case):
            x = {"n": n, "gens": _pack(_rows(g, m, n, case["gate_w"])),
                 "theta": _angles(g, m, case["theta"]),
                 "ops": _pack(_rows(g, l, n, case["op_w"])),
                 "z": _uniform(g, (case["s"],), n)}
            x["u"] = torch.randn(l, generator=g, device=DEV, dtype=torch.float64)
            out.append(x)
        return out
    n, m = case["n"], _gate_count(case)
    x = {"n": n, "m": m, "gens": _pack(_gates(g, case, n, m)),
         "theta": _angles(g, m, case["theta"])}
    if kind in ("mmd", "train"):
        x["data"] = _pack(torch.rand((case["N"], n), generator=g, device=DEV) < 0.3)
    if kind == "mmd":
        x["ops"] = _pack(torch.cat([
            torch.rand((case["per_sigma"], n), generator=g, device=DEV) < _sigma_prob(sg)
            for sg in SIGMAS]))
        l = x["ops"].shape[0]
        x["w"] = torch.full((l,), 1.0 / l, dtype=torch.float64, device=DEV)
    elif kind != "train":
        x["ops"] = _pack(_rows(g, case["l"], n, case["op_w"]))
        x["u"] = torch.randn(case["l"], generator=g, device=DEV, dtype=torch.float64)
    if kind == "indep":
        x["z"] = _uniform(g, (case["l"], case["s"]), n)
    elif kind not in ("bitflip", "train"):
        x["z"] = _uniform(g, (case["s"],), n)
    return x


def prepare(case, seed):
    x = _inputs(case, seed)
    kind = case["kind"]
    state = {"kind": kind, "case": case}
    if kind == "batch":
        probs = [(Circuit(p["n"], p["gens"], p["theta"]), p["ops"], p["z"]) for p in x]
        state.update(plan=BatchPlan(probs, case["prec"]), u=[p["u"] for p in x])
        return state
    state.update(x)
    if kind == "expval":
        state["circ"] = Circuit(x["n"], x["gens"], x["theta"])
    elif kind == "indep":
        state["circ"] = Circuit(x["n"], x["gens"], x["theta"])
    elif kind in ("grad", "mmd", "bitflip"):
        state["theta"] = x["theta"].requires_grad_(True)
    else:  # train
        m = x["m"]
        state["trainer"] = Trainer(
            x["n"], x["gens"], np.arange(m), m, x["data"], [case["per_sigma"]] * len(SIGMAS),
            [_sigma_prob(sg) for sg in SIGMAS], case["s"], precision=case["prec"], lr=1e-3,
            seed=(seed, 2), group_precision="auto" if case["auto"] else None)
        state["params"] = x["theta"].clone()
    return state


def run(st):
    kind, case = st["kind"], st["case"]
    if kind == "expval":
        mean, se, _ = iqp_expval(st["circ"], st["ops"], st["z"], case["prec"])
        return {"mean": mean, "stderr": se}
    if kind == "grad":
        mean, se = IQPExpval.apply(st["theta"], st["gens"], st["ops"], st["z"], st["n"],
                                   case["prec"])
        (g,) = torch.autograd.grad(mean, st["theta"], st["u"])
        return {"mean": mean.detach(), "stderr": se, "grad": g}
    if kind == "mmd":
        loss = IQPMMDLoss.apply(st["theta"], st["gens"], st["ops"], st["w"], st["z"], st["data"],
                                st["n"], True, case["prec"])
        (g,) = torch.autograd.grad(loss, st["theta"])
        return {"loss": loss.detach(), "grad": g}
    if kind == "batch":
        means, ses = st["plan"].expval()
        grads = st["plan"].expval_grad(st["u"])
        return {"mean": list(means), "stderr": list(ses), "grad": list(grads)}
    if kind == "indep":
        mean, se, ph = iqp_expval_indep(st["circ"], st["ops"], st["z"], phase_save=True)
        g = iqp_expval_indep_grad(st["circ"], st["ops"], st["z"], st["u"], ph)
        return {"mean": mean, "stderr": se, "grad": g}
    if kind == "bitflip":
        mean = IQPBitflipExpval.apply(st["theta"], st["gens"], st["ops"], st["n"])
        (g,) = torch.autograd.grad(mean, st["theta"], st["u"])
        return {"mean": mean.detach(), "grad": g}
    tr = st["trainer"]
    loss = tr.step(st["params"], 1)
    return {"loss": loss, "grad": tr.grad, "params": st["params"]}


# --- work -----------------------------------------------------------------------
def _odd(w, v, n):
    """P(|a and b| odd) for strings of weights w and v on n qubits (weight 0
    standing for Bernoulli(3/n) bits), by independent bits."""
    def bit(x):
        return 3.0 / n if x == 0 else (abs(x) if x < 0 else (1 + min(x, n)) / 2.0) / n
    return (1.0 - (1.0 - 2.0 * bit(v)) ** (bit(w) * n)) / 2.0


def _one_work(n, m, l, s, d, dirs, z_rows=None):
    """Bit rows and angles in, results out; two operations for every
    (observable, sample, anticommuting gate) term and direction."""
    W8 = (n + 63) // 64 * 8
    b = (m + l + (s if z_rows is None else z_rows)) * W8 + 8.0 * m + 16.0 * l
    if dirs == 2:
        b += 8.0 * m + 8.0 * l
    return b, 2.0 * dirs * l * s * m * d


def work(case):
    kind = case["kind"]
    if kind == "batch":
        b = f = 0.0
        for n, m, l in _shapes(case):
            x, y = _one_work(n, m, l, case["s"], _odd(case["gate_w"], case["op_w"], n), 2)
            b, f = b + x, f + y
        return {"bytes": b, "flops": f}
    n, m, s = case["n"], _gate_count(case), case.get("s", 1)
    gw = -2 if case.get("local") else case["gate_w"]
    if kind in ("mmd", "train"):
        b = f = 0.0
        for sg in SIGMAS:
            d = (1.0 - (1.0 - 2.0 * _sigma_prob(sg)) ** 2) / 2.0
            x, y = _one_work(n, m, case["per_sigma"], s, d, 2)
            b, f = b + x, f + y
        W8 = (n + 63) // 64 * 8
        b += case["N"] * W8 - 2 * (m * (W8 + 16) + s * W8)
        return {"bytes": b + (24.0 * 2 * m if kind == "train" else 0.0), "flops": f}
    l = case["l"]
    d = _odd(gw, case["op_w"], n)
    dirs = 1 if kind == "expval" else 2
    b, f = _one_work(n, m, l, s if kind != "bitflip" else 1, d, dirs,
                     l * s if kind == "indep" else (0 if kind == "bitflip" else None))
    return {"bytes": b, "flops": f}


# --- the same in 64 bits ----------------------------------------------------------
def _bits(words, n):
    q = torch.arange(64, device=words.device)
    b = (words.unsqueeze(-1) >> q) & 1
    return b.reshape(*words.shape[:-1], -1)[..., :n].to(torch.float32)


def _parity(a, b):
    """Parities of 0/1 float rows a against b, as float32 (counts are exact)."""
    return torch.remainder(a @ b.T, 2.0)


def _estimate(x, z, weights=None, u=None):
    """(mean, stderr, grad) of the estimator; with ``u`` the gradient of
    sum u mean, with ``weights(csum) -> (alpha, beta)`` that of a loss with
    dL/dcos = alpha + beta cos."""
    n = x["n"]
    G, A, Z = _bits(x["gens"], n), _bits(x["ops"], n), _bits(z, n)
    th = x["theta"].detach()
    s, m, l = Z.shape[0], G.shape[0], A.shape[0]
    C = _parity(A, G).to(torch.float64)
    Cth = C * (2.0 * th)
    step = max(256, int(3e8 // m))
    c1 = torch.zeros(l, dtype=torch.float64, device=DEV)
    c2 = torch.zeros_like(c1)
    E = torch.empty((l, s), dtype=torch.float64, device=DEV)
    for i in range(0, s, step):
        B = 1.0 - 2.0 * _parity(Z[i:i + step], G).to(torch.float64)
        E[:, i:i + step] = Cth @ B.T
        co = torch.cos(E[:, i:i + step])
        c1 += co.sum(1)
        c2 += (co * co).sum(1)
    del Cth
    mean = c1 / s
    se = torch.sqrt(torch.clamp(c2 / s - mean * mean, min=0.0) / s)
    if weights is not None:
        al, be = weights(c1, c2)
    elif u is not None:
        al, be = u / s, torch.zeros_like(u)
    else:
        return mean, se, None, c1, c2
    grad = torch.zeros(m, dtype=torch.float64, device=DEV)
    for i in range(0, s, step):
        e = E[:, i:i + step]
        S = (al[:, None] + be[:, None] * torch.cos(e)) * torch.sin(e)
        B = 1.0 - 2.0 * _parity(Z[i:i + step], G).to(torch.float64)
        T = S.T.contiguous() @ C
        grad -= 2.0 * (T * B).sum(0)
    return mean, se, grad, c1, c2


def _mmd(x, z, ops, w):
    n = x["n"]
    s, N = z.shape[0], x["data"].shape[0]
    sv = (1.0 - 2.0 * _parity(_bits(ops, n), _bits(x["data"], n)).to(torch.float64)).sum(1)
    p = sv / N

    def weights(c1, c2):
        d = s * (s - 1.0)
        return w * (-2.0 * p / s + 2.0 * c1 / d), -2.0 * w / d

    y = dict(x, ops=ops)
    _, _, grad, c1, c2 = _estimate(y, z, weights=weights)
    q = c1 / s
    P2 = (sv * sv - N) / (N * (N - 1.0))
    Q2 = (c1 * c1 - c2) / (s * (s - 1.0))
    return (w * (P2 - 2.0 * p * q + Q2)).sum(), grad


def _philox(seed, step, tag, count):
    """The first ``count`` outputs of the Philox4x64-10 stream (seed, step, tag)."""
    ctr = (step << 64) + (tag << 128) - 1  # numpy increments before each block
    ctr %= 1 << 256
    words = [(ctr >> (64 * i)) & (2 ** 64 - 1) for i in range(4)]
    bg = np.random.Philox(counter=np.array(words, dtype=np.uint64),
                          key=np.array(seed, dtype=np.uint64))
    return bg.random_raw(count)


def exact(case, seed):
    kind = case["kind"]
    x = _inputs(case, seed)
    if kind == "batch":
        out = {"mean": [], "stderr": [], "grad": []}
        for p in x:
            mean, se, g, _, _ = _estimate(p, p["z"], u=p["u"])
            for k, v in (("mean", mean), ("stderr", se), ("grad", g)):
                out[k].append(v)
        return out
    n = x["n"]
    if kind == "expval":
        mean, se, _, _, _ = _estimate(x, x["z"])
        return {"mean": mean, "stderr": se}
    if kind == "grad":
        mean, se, g, _, _ = _estimate(x, x["z"], u=x["u"])
        return {"mean": mean, "stderr": se, "grad": g}
    if kind == "mmd":
        loss, g = _mmd(x, x["z"], x["ops"], x["w"])
        return {"loss": loss, "grad": g}
    if kind == "bitflip":
        C = _parity(_bits(x["ops"], n), _bits(x["gens"], n)).to(torch.float64)
        c = torch.cos(2.0 * x["theta"])
        mean = torch.exp(C @ torch.log(torch.abs(c)))
        mean = mean * (1.0 - 2.0 * torch.remainder(C @ (c < 0).to(torch.float64), 2.0))
        g = -2.0 * torch.tan(2.0 * x["theta"]) * (C.T @ (x["u"] * mean))
        return {"mean": mean, "grad": g}
    if kind == "indep":
        G, A = _bits(x["gens"], n), _bits(x["ops"], n)
        C = _parity(A, G)
        l, s = case["l"], case["s"]
        mean = torch.empty(l, dtype=torch.float64, device=DEV)
        se = torch.empty_like(mean)
        grad = torch.zeros(G.shape[0], dtype=torch.float64, device=DEV)
        for k in range(l):
            J = torch.nonzero(C[k]).flatten()
            B = 1.0 - 2.0 * _parity(_bits(x["z"][k], n), G[J]).to(torch.float64)
            e = B @ (2.0 * x["theta"][J])
            co = torch.cos(e)
            mean[k] = co.mean()
            se[k] = torch.sqrt(torch.clamp((co * co).mean() - mean[k] ** 2, min=0.0) / s)
            grad[J] += -2.0 / s * x["u"][k] * (torch.sin(e) @ B)
        return {"mean": mean, "stderr": se, "grad": grad}
    # train: the first step's draws are the Philox streams of the seed
    per, W = case["per_sigma"], (n + 63) // 64
    l, s = per * len(SIGMAS), case["s"]
    z = torch.from_numpy(_philox((seed, 2), 0, 0, s * W).view(np.int64).reshape(s, W)).to(DEV)
    if n % 64:
        z[:, -1] &= (1 << (n % 64)) - 1
    raw = _philox((seed, 2), 0, 1, l * n).reshape(l, n)
    limit = np.repeat(np.array([math.floor(_sigma_prob(sg) * 2.0 ** 64) for sg in SIGMAS],
                               dtype=np.uint64), per)
    ops = _pack(torch.from_numpy(raw < limit[:, None]).to(DEV))
    w = torch.full((l,), 1.0 / l, dtype=torch.float64, device=DEV)
    loss, g = _mmd(x, z, ops, w)
    # Adam's first step: both bias-corrected moments are those of g itself
    params = x["theta"] - 1e-3 * g / (torch.abs(g) + 1e-8)
    return {"loss": loss.reshape(1), "grad": g, "params": params}
