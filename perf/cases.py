"""Performance cases of the multi-marginal Sinkhorn library.

Every case is one call sequence of a program that uses the package: a plan is at hand, its
scaling vectors are reset, a number of sweeps runs and the scaling vectors are taken.  The
cases cover the four product paths (FP64 and mixed direct sums, truncated sums, NFFT fast
summation, dense and row-by-row NFFT circles), the batched form and solving a problem that
was not seen before.  `exact` repeats the same iterations in FP64 with plain torch.

Scaling vectors come out of the library as doubles.  The FP64 paths are taken as they are;
the mixed and 16-bit paths hold six to seven digits, and the program keeps those in FP32.
"""
import math

import numpy as np
import torch

from paper_2208_03120_amd import mot, workloads as W

PATH = {"direct": mot.DIRECT, "nfft": mot.NFFT, "trunc": mot.TRUNC, "dense": mot.DENSE}
PREC = {"fp64": mot.PREC_FP64, "mixed": mot.PREC_MIXED, "bf16": mot.PREC_BF16, "fp16": mot.PREC_FP16,
        "bf16x3": mot.PREC_BF16X3}


def listed():
    return [
        # the smallest solve of the benchmark: three marginals of 500 points in FP64, where
        # the launches of a sweep and their latency count
        {"name": "path_fp64_n500", "kind": "tree", "shape": "chain", "K": 3, "n": 500, "spread": 1.0, "d": 2,
         "eta": 0.1, "path": "direct", "prec": "fp64", "sweeps": 100},
        # a reference solution in FP64 on a branching tree with ragged marginals
        {"name": "tree_fp64_n7000", "kind": "tree", "shape": "prufer", "K": 5, "n": 7000, "spread": 1.6, "d": 3,
         "eta": 0.05, "path": "direct", "prec": "fp64", "sweeps": 10},
        # the plain O(N^2) path at the headline's size
        {"name": "star_direct_n100000", "kind": "tree", "shape": "star", "K": 10, "n": 100000, "spread": 1.0, "d": 3,
         "eta": 0.05, "path": "direct", "prec": "mixed", "sweeps": 2},
        # the headline: star tree, 3-D, fixed grid and cutoff
        {"name": "star_nfft_n100000", "kind": "tree", "shape": "star", "K": 10, "n": 100000, "spread": 1.0, "d": 3,
         "eta": 0.05, "path": "nfft", "prec": "mixed", "sweeps": 10, "M": 32, "grid": 128, "m": 6},
        # small eta, where the products are truncated sums over a cell list
        {"name": "star_trunc_n100000", "kind": "tree", "shape": "star", "K": 10, "n": 100000, "spread": 1.0, "d": 3,
         "eta": 1e-3, "path": "trunc", "prec": "mixed", "sweeps": 4},
        # an ordinary tree: ragged marginals, parameters chosen by the library
        {"name": "tree_nfft_n6000", "kind": "tree", "shape": "prufer", "K": 7, "n": 6000, "spread": 2.0, "d": 3,
         "eta": 0.08, "path": "nfft", "prec": "mixed", "sweeps": 20},
        # a generalised barycenter in 2-D: weighted edges, free inner nodes, its marginals
        {"name": "barycenter_n5000", "kind": "bary", "n": 5000, "eta": 5e-3, "path": "nfft", "prec": "mixed",
         "sweeps": 20},
        # the circle at the benchmark's size, the accurate dense products
        {"name": "cycle_bf16x3_n4000", "kind": "circle", "K": 5, "n": 4000, "d": 2, "eta": 0.1, "path": "dense",
         "prec": "bf16x3", "sweeps": 5},
        # the same circle row by row through the fast summation
        {"name": "cycle_nfft_n4000", "kind": "circle", "K": 5, "n": 4000, "d": 2, "eta": 0.1, "path": "nfft",
         "prec": "mixed", "sweeps": 3},
        # a small circle: a generalised Euler flow in 1-D and one of its pair marginals
        {"name": "euler_bf16x3_n400", "kind": "euler", "K": 6, "n": 400, "eta": 0.05, "sigma": "reverse",
         "path": "dense", "prec": "bf16x3", "sweeps": 50},
        # many unlike trees advanced together: d = 1, 2, 3, sizes over a factor of 50
        {"name": "batch_24", "kind": "batch", "count": 24, "n_lo": 1000, "n_hi": 50000, "sweeps": 10},
        # a problem that just arrived: points and weights on the device, plan, sweeps, result
        {"name": "new_tree_n20000", "kind": "new", "shape": "prufer", "K": 4, "n": 20000, "spread": 1.0, "d": 2,
         "eta": 0.05, "path": "nfft", "prec": "mixed", "sweeps": 50},
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    kind = rng.choice(["fp64", "direct", "nfft", "nfft", "trunc", "bary", "dense", "dense", "cnfft", "euler", "batch",
                       "new"])
    shape = rng.choice(["chain", "star", "prufer"])
    c = {"kind": "tree", "shape": shape, "K": rng.randint(3, 12), "spread": rng.uniform(1.0, 2.5),
         "d": rng.randint(1, 3)}
    if kind == "fp64":
        c.update(K=rng.randint(2, 6), n=int(_log(rng, 100, 7000)), eta=_log(rng, 0.02, 0.3), path="direct",
                 prec="fp64", sweeps=rng.randint(5, 20))
    elif kind == "direct":
        c.update(n=int(_log(rng, 300, 40000)), eta=_log(rng, 5e-3, 0.3), path="direct", prec="mixed", sweeps=4)
    elif kind == "nfft":
        c.update(n=int(_log(rng, 500, 100000)), eta=_log(rng, 0.02, 0.3), path="nfft", prec="mixed",
                 sweeps=rng.randint(5, 20))
    elif kind == "trunc":
        c.update(d=rng.randint(2, 3), n=int(_log(rng, 5000, 60000)), eta=_log(rng, 3e-4, 3e-3), path="trunc",
                 prec="mixed", sweeps=4)
    elif kind == "bary":
        c = {"kind": "bary", "n": int(_log(rng, 400, 6000)), "eta": _log(rng, 4e-3, 2e-2), "path": "nfft",
             "prec": "mixed", "sweeps": rng.randint(5, 20)}
    elif kind == "dense":
        c = {"kind": "circle", "K": rng.randint(3, 7), "n": int(_log(rng, 60, 4500)), "d": rng.randint(1, 3),
             "eta": _log(rng, 0.03, 0.3), "path": "dense", "prec": rng.choice(["bf16x3", "bf16", "fp16"]),
             "sweeps": 5}
    elif kind == "cnfft":
        c = {"kind": "circle", "K": rng.randint(3, 5), "n": int(_log(rng, 100, 3000)), "d": rng.randint(1, 2),
             "eta": _log(rng, 0.05, 0.3), "path": "nfft", "prec": "mixed", "sweeps": 3}
    elif kind == "euler":
        c = {"kind": "euler", "K": rng.randint(4, 8), "n": int(_log(rng, 100, 1500)), "eta": _log(rng, 0.04, 0.1),
             "sigma": rng.choice(["reverse", "tent"]), "path": "dense", "prec": "bf16x3", "sweeps": rng.randint(5, 50)}
    elif kind == "batch":
        c = {"kind": "batch", "count": rng.randint(4, 24), "n_lo": rng.randint(300, 2000),
             "n_hi": int(_log(rng, 4000, 40000)), "sweeps": rng.randint(3, 10)}
    else:
        c.update(kind="new", K=rng.randint(3, 6), n=int(_log(rng, 500, 40000)), eta=_log(rng, 0.03, 0.2),
                 path="nfft", prec="mixed", sweeps=rng.randint(10, 50))
    return c


def _rng(seed):
    return np.random.Generator(np.random.PCG64(int(seed)))


def _instances(case, seed):
    """The case's problems: a list of (instance, edge weights, free flags, closing points)."""
    rng = _rng(seed)
    kind = case["kind"]
    if kind in ("tree", "new"):
        K = case["K"]
        parent = {"chain": W.chain_parent, "star": W.star_parent}.get(case["shape"])
        # the topology goes with the case; points, weights and ragged sizes with the seed
        parent = parent(K) if parent else W.prufer_parent(_rng(1000 + K), K)
        # ragged marginals around n: factors spread over [1 / spread, 1]
        shape = _rng(7 + K).uniform(1.0 / case["spread"], 1.0, size=K)
        sizes = [max(2, int(case["n"] * f)) if case["spread"] > 1.0 else case["n"] for f in shape]
        return [(W.make_instance(rng, K, sizes, case["d"], W.TREE, case["eta"], parent=parent), None, None, None)]
    if kind == "bary":
        inst, ew, free = W.h_tree_barycenter(seed=seed, N=case["n"], eta=case["eta"])
        return [(inst, ew, free, None)]
    if kind == "circle":
        return [(W.make_instance(rng, case["K"], case["n"], case["d"], W.CIRCLE, case["eta"]), None, None, None)]
    if kind == "euler":
        inst, closing = W.euler_flow(seed=seed, N=case["n"], K=case["K"], eta=case["eta"], sigma=case["sigma"])
        return [(inst, None, None, closing)]
    got = []
    for i in range(case["count"]):
        r = _rng(4 + i)  # topology, sizes, dimension and eta of the i-th member of the batch
        K = int(r.integers(3, 13))
        n = int(round(math.exp(r.uniform(math.log(case["n_lo"]), math.log(case["n_hi"])))))
        d = int(r.integers(1, 4))
        parent = W.prufer_parent(r, K)
        eta = float(r.uniform(0.02, 0.2))
        got.append((W.make_instance(rng, K, n, d, W.TREE, eta, parent=parent, weights="dirichlet"), None, None, None))
    return got


def _plan(case, problem):
    inst, ew, free, closing = problem
    fs = mot.fastsum_params(M=case["M"], n=case["grid"], m=case["m"]) if "grid" in case else None
    return mot.Plan(inst.points, inst.weights, inst.topology, inst.parent, inst.eta,
                    path=PATH[case.get("path", "nfft")], precision=PREC[case.get("prec", "mixed")], fastsum=fs,
                    edge_weight=ew, free=free, closing_points=closing)


def _dtype(case):
    return torch.float64 if case.get("prec") == "fp64" else torch.float32


def prepare(case, seed):
    problems = _instances(case, seed)
    state = {"case": case, "dtype": _dtype(case)}
    if case["kind"] == "new":  # the problem only: the plan is part of the pass
        inst = problems[0][0]
        state["points"] = [torch.from_numpy(p).cuda() for p in inst.points]
        state["weights"] = [torch.from_numpy(w).cuda() for w in inst.weights]
        state["parent"], state["eta"] = inst.parent, inst.eta
        state["out"] = torch.empty(int(sum(inst.sizes)), dtype=torch.float64, device="cuda")
        return state
    plans = [_plan(case, p) for p in problems]
    state["plans"] = plans
    state["out"] = [torch.empty(int(p.sizes.sum()), dtype=torch.float64, device="cuda") for p in plans]
    if case["kind"] == "batch":
        state["batch"] = mot.Batch(plans)
    else:
        state["ones"] = torch.ones_like(state["out"][0])
        state["marg"] = torch.empty_like(state["out"][0])
    return state


def run(state):
    case, dtype = state["case"], state["dtype"]
    kind, sweeps = case["kind"], case["sweeps"]
    if kind == "new":
        plan = mot.Plan(state["points"], state["weights"], W.TREE, state["parent"], state["eta"],
                        path=PATH[case["path"]], precision=PREC[case["prec"]])
        _, _, S, _ = plan.sinkhorn(sweeps)
        phi = plan.scalings_device(state["out"]).to(dtype)
        plan.close()
        return {"phi": phi, "S": S}
    if kind == "batch":  # a batch sweeps on from where it stands
        state["batch"].sinkhorn(sweeps)
        return {"phi": [p.scalings_device(o).to(dtype) for p, o in zip(state["plans"], state["out"])]}
    plan = state["plans"][0]
    plan.set_scalings_device(state["ones"])
    _, _, S, _ = plan.sinkhorn(sweeps)
    got = {"phi": plan.scalings_device(state["out"][0]).to(dtype), "S": S}
    if kind == "bary":
        got["marginals"] = plan.marginals_device(state["marg"])[0].to(dtype)
    if kind == "euler":
        got["pair"] = torch.from_numpy(plan.pair_marginal(case["K"] // 2)).to(dtype)
    return got


# --- what a pass cannot do without -------------------------------------------------------

def _edges(inst):
    return [(int(inst.parent[k]), k) for k in range(1, inst.K)]


def work(case):
    nbytes = flops = 0.0
    for inst, _, _, _ in _instances(case, 1):
        sizes, d, sweeps = inst.sizes, inst.d, case["sweeps"]
        points = float(sum(sizes))
        nbytes += 8.0 * points * (d + 2)  # points and weights in, scaling vectors out
        if inst.topology == W.CIRCLE:
            K, n = inst.K, float(sizes[0])
            if case["path"] == "dense":  # 2 (K - 2) matrix products a sweep, 2 N^3 each
                flops += sweeps * 2.0 * (K - 2) * 2.0 * n ** 3
            else:  # one fast summation a row: window taps (2m = 10) in and out
                flops += sweeps * 2.0 * (K - 2) * n * 2.0 * (2.0 * n * 10.0 ** d)
            nbytes += sweeps * 2.0 * (K - 2) * 2.0 * n * n * 4.0  # a product's matrix in and out
            continue
        nbytes += sweeps * 8.0 * points * 5.0  # mu, phi in and out, the messages in and out
        for p, k in _edges(inst):
            if case.get("path", "nfft") == "nfft":
                taps = (2.0 * case.get("m", 5)) ** d
                flops += sweeps * 2.0 * 2.0 * taps * (sizes[p] + sizes[k])
            else:
                pairs = float(sizes[p]) * sizes[k]
                if case["path"] == "trunc":  # the cutoff ball's share of the cloud's box
                    rc = math.sqrt(case["eta"] * math.log(1e9))
                    ball = {1: 2.0 * rc, 2: math.pi * rc ** 2, 3: 4.0 / 3.0 * math.pi * rc ** 3}[d]
                    pairs *= min(1.0, ball / 0.5 ** d)
                # differences, squares, exponential (one operation) and weighted sum
                flops += sweeps * 2.0 * pairs * (3.0 * d + 3.0)
    return {"bytes": nbytes, "flops": flops}


# --- the same iterations in FP64, plain torch --------------------------------------------

def _apply(x, y, eta, v, block=1 << 28):
    """sum_j v_j exp(-|x_i - y_j|^2 / eta), rows in blocks."""
    ctr = y.mean(0)
    x, y = x - ctr, y - ctr
    xs = torch.cat([2.0 * x / eta, -(x * x).sum(1, keepdim=True) / eta, torch.ones_like(x[:, :1])], 1)
    ys = torch.cat([y, torch.ones_like(y[:, :1]), -(y * y).sum(1, keepdim=True) / eta], 1).T.contiguous()
    step = max(1, block // y.shape[0])
    return torch.cat([torch.mv((xs[i:i + step] @ ys).exp_(), v) for i in range(0, x.shape[0], step)])


def _exact_tree(inst, ew, free, sweeps, want_marginals=False):
    X = [torch.from_numpy(p).cuda() for p in inst.points]
    mu = [None if w is None else torch.from_numpy(w).cuda() for w in inst.weights]
    K, parent = inst.K, inst.parent
    eta = [inst.eta / (1.0 if ew is None else float(ew[k])) for k in range(K)]
    kids = [[c for c in range(1, K) if parent[c] == k] for k in range(K)]
    phi = [torch.ones(len(x), dtype=torch.float64, device="cuda") for x in X]
    beta, gamma = [None] * K, [None] * K

    def prod(k, but=-1):
        out = torch.ones_like(phi[k])
        for c in kids[k]:
            if c != but:
                out = out * beta[c]
        return out

    def up():
        for k in range(K - 1, 0, -1):
            beta[k] = _apply(X[parent[k]], X[k], eta[k], phi[k] * prod(k))

    def down(k):
        p = parent[k]
        src = phi[p] * prod(p, k) * (gamma[p] if p > 0 else 1.0)
        gamma[k] = _apply(X[k], X[p], eta[k], src)

    up()
    S = 0.0
    for _ in range(sweeps):
        S = 0.0
        for k in range(K):
            if k > 0:
                down(k)
            if free is not None and free[k]:
                continue
            old = phi[k]
            phi[k] = mu[k] / (prod(k) * (gamma[k] if k > 0 else 1.0))
            at = mu[k] > 0
            S += float((mu[k][at] * torch.log(old[at])).sum())
            if k == 0:
                S -= float((mu[0][at] / phi[0][at] * old[at]).sum())
        up()
    got = {"phi": torch.cat(phi), "S": inst.eta * S}
    if want_marginals:
        P = []
        for k in range(K):
            if k > 0:
                down(k)
            P.append(phi[k] * prod(k) * (gamma[k] if k > 0 else 1.0))
        got["marginals"] = torch.cat(P)
    return got


def _exact_circle(inst, closing, sweeps, pair=0):
    X = [torch.from_numpy(p).cuda() for p in inst.points]
    mu = [torch.from_numpy(w).cuda() for w in inst.weights]
    K = inst.K

    def kmat(a, b):
        d2 = sum((a[:, None, c] - b[None, :, c]) ** 2 for c in range(inst.d))
        return torch.exp(-d2 / inst.eta)

    edge = [kmat(X[k], X[k + 1]) for k in range(K - 1)]  # K^{(k, k+1)}
    close = kmat(X[0] if closing is None else torch.from_numpy(closing).cuda(), X[K - 1])
    phi = [torch.ones(len(x), dtype=torch.float64, device="cuda") for x in X]
    beta = [None] * K  # beta[k]: n_0 x n_k, the chain from k on to the closing edge
    beta[K - 1] = close

    def up():
        for k in range(K - 2, 0, -1):
            beta[k] = (beta[k + 1] * phi[k + 1]) @ edge[k].T.contiguous()

    def gammas():  # n_0 x n_k: the chain from 0 to k
        g = edge[0]
        yield 1, g
        for k in range(2, K):
            g = (g * phi[k - 1]) @ edge[k - 1]
            yield k, g

    up()
    S = 0.0
    for _ in range(sweeps):
        old = phi[0]
        phi[0] = mu[0] / torch.mv(edge[0] * beta[1], phi[1])
        S = float((mu[0] * torch.log(old)).sum() - (mu[0] / phi[0] * old).sum())
        for k, g in gammas():
            old = phi[k]
            phi[k] = mu[k] / torch.mv((beta[k] * g).T.contiguous(), phi[0])
            S += float((mu[k] * torch.log(old)).sum())
        up()
    got = {"phi": torch.cat(phi), "S": inst.eta * S}
    if pair:
        for k, g in gammas():
            if k == pair:
                got["pair"] = phi[0][:, None] * g * beta[k] * phi[k]
    return got


def exact(case, seed):
    problems = _instances(case, seed)
    if case["kind"] == "batch":
        return {"phi": [_exact_tree(p[0], None, None, case["sweeps"])["phi"] for p in problems]}
    inst, ew, free, closing = problems[0]
    if inst.topology == W.CIRCLE:
        return _exact_circle(inst, closing, case["sweeps"], case["K"] // 2 if case["kind"] == "euler" else 0)
    return _exact_tree(inst, ew, free, case["sweeps"], case["kind"] == "bary")
