"""Timed cases of the maximum common induced subgraph framework.

Each case is one of the calls that a program makes: `solve_batch` on pairs it
has just read (host graphs in, results out), a `Plan` kept on the GPU and run
again (the batched service loop), `solve_goals`, a search ordered by the
learned policy, and the policy's own forward and training steps.

Search outputs are each pair's size and proof flag.  The mapping itself is
returned only where there is just one (a relabelled copy of an asymmetric
graph): elsewhere several largest mappings exist and the parallel search
reports whichever it met first.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1908_06418_amd import Plan, solve, solve_batch, solve_goals
from paper_1908_06418_amd.policy import Policy

F, HID = 16, 64                      # the policy network: 16 -> 64 -> 64 -> 1
N_PARAMS = HID * F + HID + HID * HID + HID + HID + 1


def listed():
    return [
        # A program that asks for one small pair after another, each call with
        # its own results: latency.
        {"name": "pairs_n16", "do": "one_by_one", "count": 8, "n0": 12, "n1": 18, "p0": 0.3, "p1": 0.3},
        # The same near the top of the paper's small band (fewer than 40
        # vertices): a single search tree at a time, spread over the GPU.
        {"name": "pairs_n30", "do": "one_by_one", "count": 6, "n0": 27, "n1": 30, "p0": 0.3, "p1": 0.3},
        # A batch of many small pairs of mixed size and density, solved once
        # (marshalling, ordering, upload and results are part of the call).
        {"name": "batch_4096", "do": "solve", "count": 4096, "n0": 10, "n1": 22, "p0": 0.1, "p1": 0.5},
        # The batched service loop on resident inputs: harder pairs, replayed
        # as a HIP graph.  Throughput of the search kernel on 32-bit rows.
        {"name": "plan_60_n30", "do": "plan", "count": 60, "n0": 30, "n1": 30, "p0": 0.1, "p1": 0.5},
        # The same on 64-bit rows: pairs of up to 33 vertices.
        {"name": "plan_256_n33", "do": "plan", "count": 256, "n0": 10, "n1": 33, "p0": 0.1, "p1": 0.35},
        # Directed vertex-labelled pairs (chemical or workflow graphs), once.
        {"name": "directed_labelled_60", "do": "solve", "count": 60, "n0": 40, "n1": 60, "p0": 0.1, "p1": 0.1,
         "directed": True, "labels": 0.33},
        # The same kind beyond 64 vertices (128-bit rows).
        {"name": "directed_labelled_100", "do": "plan", "count": 40, "n0": 80, "n1": 100, "p0": 0.1, "p1": 0.1,
         "directed": True, "labels": 0.33},
        # Labelled pairs up to the vertex limit (256-bit rows).
        {"name": "labelled_254", "do": "plan", "count": 16, "n0": 129, "n1": 254, "p0": 0.5, "p1": 0.5,
         "labels": 0.66},
        # Isomorphism through the same call: a graph and a relabelled copy.
        {"name": "copies_254", "do": "copies", "count": 8, "n0": 129, "n1": 254, "p0": 0.2, "p1": 0.2},
        # A search whose shallow nodes are ordered by the learned policy.
        {"name": "learned_24_n28", "do": "plan", "count": 24, "n0": 28, "n1": 28, "p0": 0.2, "p1": 0.4,
         "learned": True},
        # Training the policy: gradient and update on as many rows as the
        # stored training traces hold.
        {"name": "policy_step_41358", "do": "step", "rows": 41358},
        # Scoring a large set of candidate rows.
        {"name": "policy_forward_1m", "do": "forward", "rows": 1000000},
    ]


def _between(rng, lo, hi):
    """A whole number of [lo, hi], spread over its logarithm."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(("pair", "batch", "plan", "labelled", "wide", "copies", "goals", "learned",
                       "forward", "step"))
    if kind == "pair":
        n, p = rng.randint(8, 29), round(rng.uniform(0.1, 0.5), 3)
        return {"do": "one_by_one", "count": rng.randint(6, 12), "n0": max(2, n - 6), "n1": n, "p0": p, "p1": p}
    if kind == "batch":
        n = rng.randint(12, 22)
        return {"do": "solve", "count": _between(rng, 8, 4096), "n0": rng.randint(2, n), "n1": n,
                "p0": 0.1, "p1": 0.5, "ordering": rng.choice(("degree", "degree", "btf", "portfolio"))}
    if kind == "plan":
        n = rng.randint(20, 33)
        return {"do": "plan", "count": _between(rng, 8, 60 if n <= 30 else 256), "n0": n if n <= 30 else 10,
                "n1": n, "p0": 0.1, "p1": 0.5 if n <= 30 else 0.35}
    if kind == "labelled":
        n = rng.randint(33, 64)
        return {"do": rng.choice(("solve", "plan")), "count": _between(rng, 6, 256), "n0": rng.randint(20, n),
                "n1": n, "p0": 0.1, "p1": 0.1, "directed": rng.random() < 0.7, "labels": 0.5}
    if kind == "wide":
        n = rng.randint(65, 254)
        return {"do": "plan", "count": _between(rng, 6, 40), "n0": (n + 1) // 2, "n1": n,
                "p0": 0.1 if n <= 128 else 0.5, "p1": 0.1 if n <= 128 else 0.5,
                "directed": n <= 100 and rng.random() < 0.5, "labels": 0.75}
    if kind == "copies":
        n = rng.randint(40, 254)
        return {"do": "copies", "count": _between(rng, 4, 32), "n0": max(40, n // 2), "n1": n, "p0": 0.2, "p1": 0.2}
    if kind == "goals":
        n = rng.randint(16, 30)
        return {"do": "goals", "count": _between(rng, 6, 20), "n0": n, "n1": n, "p0": 0.1, "p1": 0.1,
                "strategy": rng.choice(("top-down", "bisect"))}
    if kind == "learned":
        n = rng.randint(16, 28)
        return {"do": "plan", "count": _between(rng, 6, 24), "n0": n, "n1": n, "p0": 0.2, "p1": 0.4, "learned": True}
    if kind == "forward":
        return {"do": "forward", "rows": _between(rng, 1, 1 << 20)}
    return {"do": "step", "rows": _between(rng, 1, 1 << 18)}


# ---- inputs ----------------------------------------------------------------

def _graph_of(a, label):
    rows = np.packbits(a, axis=1, bitorder="little")
    return {"n": a.shape[0], "directed": False, "rows": [int.from_bytes(r.tobytes(), "little") for r in rows],
            "label": label}


def _matrix(rng, n, p, directed):
    a = rng.random((n, n)) < p
    if not directed:
        a = np.triu(a, 1)
        a = a | a.T
    np.fill_diagonal(a, False)
    return a


def _pairs(case, seed):
    """Random pairs G(n, p), n and p shared by the two graphs of a pair; for
    "copies", the second graph is the first one relabelled.  Also returns the
    relabelling of each copy (vertex i of G is vertex perm[i] of H)."""
    rng = np.random.default_rng([seed, 1])
    directed, labels = bool(case.get("directed")), case.get("labels", 0)
    out, perms = [], []
    for i in range(case["count"]):
        n = int(rng.integers(case["n0"], case["n1"] + 1))
        if case["do"] == "copies":  # sizes evenly over the range
            n = case["n0"] + (case["n1"] - case["n0"]) * i // max(1, case["count"] - 1)
        p = rng.uniform(case["p0"], case["p1"])
        pair = []
        for side in range(2):
            if case["do"] == "copies" and side:
                perm = rng.permutation(n)
                b = np.zeros_like(a)
                b[np.ix_(perm, perm)] = a
                perms.append(perm)
                a = b
            else:
                a = _matrix(rng, n, p, directed)
            label = rng.integers(0, max(1, math.ceil(labels * n)), n).tolist() if labels else None
            g = _graph_of(a, label)
            g["directed"] = directed
            pair.append(g)
        out.append(tuple(pair))
    return out, perms


def _params(seed):
    """A random start of the policy network, packed W1, b1, W2, b2, w3, b3."""
    rng = np.random.default_rng([seed, 2])
    return np.concatenate([rng.normal(0, math.sqrt(2 / F), HID * F), rng.normal(0, 0.1, HID),
                           rng.normal(0, math.sqrt(2 / HID), HID * HID), rng.normal(0, 0.1, HID),
                           rng.normal(0, math.sqrt(1 / HID), HID), rng.normal(0, 0.1, 1)]).astype(np.float32)


def _rows(rows, seed):
    """Candidate rows as the search sees them (16 features: shares of n, two
    flags and a constant one) and their labels."""
    rng = np.random.default_rng([seed, 3])
    x = rng.random((rows, F), dtype=np.float32)
    x[:, 12] = rng.integers(0, 2, rows)
    x[:, 13] = rng.random(rows) < 0.2
    x[:, 14] = 0
    x[:, 15] = 1
    y = (rng.random(rows) < 0.3).astype(np.float32)
    return x.astype(np.float16), y


LEARNING_RATE = 0.5


def prepare(case, seed):
    if case["do"] in ("forward", "step"):
        x, y = _rows(case["rows"], seed)
        return {"do": case["do"], "policy": Policy(_params(seed)), "x": torch.from_numpy(x).cuda(),
                "y": torch.from_numpy(y).cuda()}
    pairs, _ = _pairs(case, seed)
    state = {"do": case["do"], "pairs": pairs, "ordering": case.get("ordering", "degree"),
             "strategy": case.get("strategy")}
    if case["do"] == "plan":
        # the plan, its workspace and its policy stay with such a program
        state["plan"] = Plan(pairs, tuning={"use_graph": 1},
                             policy=Policy(_params(seed)) if case.get("learned") else None).upload()
    return state


# ---- one pass --------------------------------------------------------------

def _sizes(results):
    return {"size": np.array([r.size for r in results], dtype=np.int32),
            "optimal": np.array([r.optimal for r in results], dtype=np.int32)}


def run(state):
    do = state["do"]
    if do == "forward":
        return state["policy"].forward(state["x"])
    if do == "step":
        policy = state["policy"]
        loss, grad = policy.grad(state["x"], state["y"])
        policy.sgd(grad, LEARNING_RATE)
        return {"loss": loss, "grad": grad, "params": policy.params.clone()}
    if do == "plan":
        state["plan"].run()
        return _sizes(state["plan"].results())
    if do == "goals":
        return _sizes(solve_goals(state["pairs"], strategy=state["strategy"]))
    if do == "one_by_one":
        return _sizes([solve(g, h) for g, h in state["pairs"]])
    results = solve_batch(state["pairs"], ordering=state["ordering"])
    out = _sizes(results)
    if do == "copies":
        out["mapping"] = np.array([gh for r in results for gh in sorted(r.mapping)], dtype=np.int32)
    return out


# ---- what a pass cannot do without ------------------------------------------

def work(case):
    if case["do"] in ("forward", "step"):
        rows = case["rows"]
        macs = F * HID + HID * HID + HID
        if case["do"] == "forward":
            return {"bytes": rows * (2 * F + 4) + 4 * N_PARAMS, "flops": 2 * rows * macs}
        # backward: the weight gradients, and the gradient through W2 and w3
        return {"bytes": rows * (2 * F + 4) + 16 * N_PARAMS,
                "flops": 2 * rows * (2 * macs + HID * HID + HID)}
    # Adjacency bits and labels in, sizes and mappings out.  The search itself
    # is integer work on data that stays on the chip; how many nodes it needs
    # depends on the inputs and is known only once it has ended.
    n = (case["n0"] + case["n1"]) / 2
    per_pair = 2 * n * 8 * math.ceil(case["n1"] / 64) + (8 * n if case.get("labels") else 0) + 8 + 8 * n
    return {"bytes": case["count"] * per_pair, "flops": 0}


# ---- the same in 64 bits -----------------------------------------------------

def exact(case, seed):
    if case["do"] in ("forward", "step"):
        return _exact_policy(case, seed)
    if case["do"] == "copies":
        # a graph and its relabelled copy: size n, by the relabelling
        _, perms = _pairs(case, seed)
        return {"size": np.array([len(p) for p in perms], dtype=np.int32),
                "optimal": np.ones(len(perms), dtype=np.int32),
                "mapping": np.concatenate([np.stack([np.arange(len(p)), p], axis=1) for p in perms]).astype(np.int32)}
    return None


def _exact_policy(case, seed):
    x, y = _rows(case["rows"], seed)
    w32 = _params(seed)
    x = torch.from_numpy(x).double()
    # the network multiplies by the weights rounded to half precision
    w = torch.from_numpy(w32).half().double()
    W1, b1, W2, b2, w3, b3 = torch.split(w, [HID * F, HID, HID * HID, HID, HID, 1])
    W1, W2 = W1.view(HID, F), W2.view(HID, HID)
    a1 = x @ W1.T + b1
    h1 = a1.clamp(min=0)
    a2 = h1 @ W2.T + b2
    h2 = a2.clamp(min=0)
    z = h2 @ w3 + b3
    if case["do"] == "forward":
        return z
    y = torch.from_numpy(y).double()
    loss = (z.clamp(min=0) - z * y + torch.log1p(torch.exp(-z.abs()))).mean()
    dz = (torch.sigmoid(z) - y) / case["rows"]
    d2 = torch.outer(dz, w3) * (a2 > 0)
    d1 = (d2 @ W2) * (a1 > 0)
    grad = torch.cat([(d1.T @ x).reshape(-1), d1.sum(0), (d2.T @ h1).reshape(-1), d2.sum(0), h2.T @ dz,
                      dz.sum().reshape(1)])
    return {"loss": loss.reshape(1), "grad": grad,
            "params": torch.from_numpy(w32).double() - LEARNING_RATE * grad}
