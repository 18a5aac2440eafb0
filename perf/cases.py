"""The calls whose speed matters to a user of this library, as cases that can be timed and compared.

A case is a dict of plain values; "path" names the entry point and the rest its sizes:

  dataset     rcd.partition_dataset on a labelled data set: route "auto" (what a user gets who asks for nothing),
              "stored" (one gain sweep over S per round), "recompute" (S never stored) or "graph_cut"
  class       rcd.partition_class on one class whose similarity matrix is at hand
  similarity  rcd.similarity, optionally of the rows that a row index picks
  bandwidth   rcd.bandwidth
  sweep       rcd.gain_sweep
  shards      rcd.worker_shards

Inputs follow the recipe of synth_inputs.py: per class a Gaussian mixture, sigma^2 = d.
"""
import math

import numpy as np
import torch

import paper_2211_00839_amd as rcd

DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16}
MODES = {"auto": rcd.MODE_AUTO, "stored": rcd.MODE_STORED, "recompute": rcd.MODE_RECOMPUTE}
CAPS_4 = "1,1,2,4"
CAPS_8 = "1,1,1,2,2,3,4,6"
CAPS_8_LARGE = "1,1,2,2,3,3,4,8"
CAPS_16 = "4,1,1,1,1,4,4,3,1,1,2,2,3,2,2,1"


def listed():
    return [
        # the smallest job: a few small classes, two equal workers; launches and per-step latency are all there is
        {"name": "tiny_auto", "path": "dataset", "route": "auto", "L": 4, "n_c": 250, "spread": 0.0, "d": 64, "dtype": "f32",
         "caps": "1,1"},
        # ten classes of 5000 (the class structure of CIFAR-10), four unequal workers, the default route
        {"name": "cifar10_auto", "path": "dataset", "route": "auto", "L": 10, "n_c": 5000, "spread": 0.0, "d": 512,
         "dtype": "f32", "caps": CAPS_4},
        # a hundred classes of 500 (CIFAR-100), sixteen workers, the default route
        {"name": "cifar100_auto", "path": "dataset", "route": "auto", "L": 100, "n_c": 500, "spread": 0.0, "d": 512,
         "dtype": "f32", "caps": CAPS_16},
        # the same job by gain sweeps over the stored similarity, the route the benchmark's headline uses
        {"name": "cifar10_sweeps", "path": "dataset", "route": "stored", "L": 10, "n_c": 5000, "spread": 0.0, "d": 512,
         "dtype": "f32", "caps": CAPS_4},
        # the graph-cut function, eight unequal workers, classes of unequal size as real data sets have them
        {"name": "hetero8_graph_cut", "path": "dataset", "route": "graph_cut", "L": 10, "n_c": 5000, "spread": 0.2, "d": 512,
         "dtype": "f32", "caps": CAPS_8},
        # no room for any similarity matrix: S is rebuilt by the matrix cores inside every sweep
        {"name": "cifar100_recompute", "path": "dataset", "route": "recompute", "L": 100, "n_c": 500, "spread": 0.0, "d": 512,
         "dtype": "f32", "caps": CAPS_16},
        # the largest: one class of 50 000 samples with its 10 GB similarity matrix, 50 000 steps
        {"name": "large_class", "path": "class", "n": 50000, "d": 2048, "dtype": "bf16", "caps": CAPS_8_LARGE},
        # one similarity build of that size
        {"name": "similarity_large", "path": "similarity", "n": 50000, "rows": 50000, "d": 2048, "dtype": "bf16"},
        # a small class picked out of a data set, with a feature length that is not a multiple of anything
        {"name": "similarity_small_ragged", "path": "similarity", "n": 601, "rows": 5000, "d": 300, "dtype": "f32"},
        # the kernel bandwidth of a data set
        {"name": "bandwidth", "path": "bandwidth", "n": 20000, "d": 512, "dtype": "f32"},
        # the gains of every candidate for every worker, one class of 5000
        {"name": "gain_sweep", "path": "sweep", "n": 5000, "K": 8},
        # the hand-off: index lists of eight workers out of a million assignments (20 classes of 50 000)
        {"name": "worker_shards", "path": "shards", "N": 1000000, "K": 8},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _caps(rng, most=16):
    return ",".join(str(rng.randint(1, 6)) for _ in range(rng.randint(2, most)))


def draw(rng):
    path = rng.choice(["dataset", "dataset", "dataset", "dataset", "class", "similarity", "similarity", "bandwidth", "sweep",
                       "shards"])
    dtype = rng.choice(["f32", "bf16"])
    if path == "dataset":
        route = rng.choice(["auto", "auto", "stored", "graph_cut", "recompute"])
        n_c = _log_int(rng, 100, 1500 if route == "recompute" else 6000)
        budget = 10000 if route == "recompute" else 50000
        L = max(1, min(_log_int(rng, 1, 100), budget // n_c))
        return {"path": path, "route": route, "L": L, "n_c": n_c, "spread": rng.choice([0.0, 0.3]),
                "d": rng.choice([64, 100, 256, 512, 777]), "dtype": dtype, "caps": _caps(rng)}
    if path == "class":
        return {"path": path, "n": _log_int(rng, 300, 40000), "d": rng.choice([128, 512]), "dtype": dtype, "caps": _caps(rng, 12)}
    if path == "similarity":
        rows = _log_int(rng, 100, 20000)
        return {"path": path, "n": max(50, int(rows * rng.choice([0.1, 0.5, 1.0]))), "rows": rows,
                "d": rng.choice([64, 100, 300, 512, 777, 1024, 2048]), "dtype": dtype}
    if path == "bandwidth":
        return {"path": path, "n": _log_int(rng, 200, 20000), "d": rng.choice([64, 300, 512, 1024]), "dtype": dtype}
    if path == "sweep":
        return {"path": path, "n": _log_int(rng, 200, 20000), "K": rng.randint(1, 16)}
    return {"path": path, "N": _log_int(rng, 1000, 1000000), "K": rng.randint(2, 16)}


def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _mixture(g, n, d, dtype, groups=4):
    centers = torch.randn(groups, d, generator=g, device="cuda")
    comp = torch.randint(0, groups, (n,), generator=g, device="cuda")
    return (centers[comp] + 0.5 * torch.randn(n, d, generator=g, device="cuda")).to(DTYPES[dtype])


def _class_sizes(case):
    """The sizes of the classes: a matter of the data set's kind, the same for every seed."""
    u = np.random.default_rng(case["L"]).uniform(-1, 1, case["L"])
    return [max(1, int(round(case["n_c"] * (1 + case["spread"] * x)))) for x in u]


def _dataset(case, seed):
    g = _gen(seed)
    sizes = _class_sizes(case)
    X = torch.cat([_mixture(g, n, case["d"], case["dtype"]) for n in sizes])
    labels = torch.cat([torch.full((n,), i, dtype=torch.int32, device="cuda") for i, n in enumerate(sizes)])
    at = torch.randperm(X.shape[0], generator=g, device="cuda")
    return X[at].contiguous(), labels[at].contiguous(), max(sizes)


def _capacities(case):
    return np.array([int(x) for x in case["caps"].split(",")], dtype=np.int32)


def prepare(case, seed):
    path = case["path"]
    s = {"case": case}
    if path == "dataset":
        s["X"], s["labels"], most = _dataset(case, seed)
        s["r"] = _capacities(case)
        mode = rcd.MODE_RECOMPUTE if case["route"] == "recompute" else rcd.MODE_STORED
        _, full = rcd.dataset_workspace_bytes(s["X"].shape[0], case["L"], most, len(s["r"]), mode)
        s["ws"] = torch.empty(full, dtype=torch.uint8, device="cuda")
    elif path == "class":
        X = _mixture(_gen(seed), case["n"], case["d"], case["dtype"], groups=8)
        s["S"] = rcd.similarity(X, float(case["d"]))
        r = _capacities(case)
        s["cap"] = rcd.quota(case["n"], r)
        s["ws"] = torch.empty(rcd.class_workspace_bytes(case["n"], len(r), rcd.MODE_INCREMENTAL), dtype=torch.uint8,
                              device="cuda")
    elif path in ("similarity", "bandwidth"):
        g = _gen(seed)
        s["X"] = _mixture(g, case.get("rows", case["n"]), case["d"], case["dtype"])
        if path == "similarity":
            s["index"] = None
            if case["rows"] != case["n"]:
                at = torch.randperm(case["rows"], generator=g, device="cuda")[: case["n"]]
                s["index"] = at.sort().values.to(torch.int32)
            s["S"] = torch.empty(case["n"], case["n"], device="cuda")
            s["ws"] = torch.empty(max(256, (case["n"] * 4 + 255) // 256 * 256), dtype=torch.uint8, device="cuda")
    elif path == "sweep":
        n, K = case["n"], case["K"]
        g = _gen(seed)
        s["S"] = rcd.similarity(_mixture(g, n, 128, "f32"), 128.0)
        # coverage after some steps: per worker the best similarity to a handful of samples, one worker still empty
        s["cur"] = torch.zeros(K, n, device="cuda")
        for k in range(1, K):
            s["cur"][k] = s["S"][torch.randint(0, n, (k,), generator=g, device="cuda")].max(0).values
        s["ws"] = torch.empty(rcd.class_workspace_bytes(n, K, rcd.MODE_STORED), dtype=torch.uint8, device="cuda")
    else:
        g = _gen(seed)
        s["assign"] = torch.randint(0, case["K"], (case["N"],), generator=g, device="cuda").to(torch.int32)
        # a few samples were left over
        s["assign"][torch.randperm(case["N"], generator=g, device="cuda")[: case["N"] // 50]] = -1
    return s


def run(s):
    case = s["case"]
    path = case["path"]
    if path == "dataset":
        if case["route"] == "graph_cut":
            assign, order, obj = rcd.partition_dataset(s["X"], s["labels"], case["L"], s["r"], float(case["d"]),
                                                       workspace=s["ws"], graph_cut=True)
        else:
            assign, order, obj = rcd.partition_dataset(s["X"], s["labels"], case["L"], s["r"], float(case["d"]),
                                                       MODES[case["route"]], s["ws"])
        return {"assign": assign, "order": order, "obj": obj}
    if path == "class":
        assign, order, obj = rcd.partition_class(S=s["S"], cap=s["cap"], workspace=s["ws"], mode=rcd.MODE_AUTO)
        return {"assign": assign, "order": order, "obj": obj}
    if path == "similarity":
        return rcd.similarity(s["X"], float(case["d"]), row_index=s["index"], out=s["S"], workspace=s["ws"])
    if path == "bandwidth":
        return rcd.bandwidth(s["X"])
    if path == "sweep":
        return rcd.gain_sweep(s["S"], s["cur"], workspace=s["ws"])
    index, offset = rcd.worker_shards(s["assign"], case["K"])
    # what the offsets leave out of the lists is nobody's and stays unwritten
    return {"index": index[: int(offset[-1])], "offset": offset}


def work(case):
    path = case["path"]
    es = 2 if case.get("dtype") == "bf16" else 4
    if path == "dataset":
        N = case["L"] * case["n_c"]
        # features, labels and outputs once; the similarities of all pairs (i < j)
        return {"bytes": N * (case["d"] * es + 12), "flops": N * case["n_c"] * case["d"]}
    if path == "class":
        return {"bytes": case["n"] ** 2 * 4 + case["n"] * 8, "flops": case["n"] ** 2}
    if path == "similarity":
        return {"bytes": case["n"] * case["d"] * es + case["n"] ** 2 * 4, "flops": case["n"] ** 2 * case["d"]}
    if path == "bandwidth":
        return {"bytes": case["n"] * case["d"] * es, "flops": case["n"] ** 2 * case["d"]}
    if path == "sweep":
        return {"bytes": case["n"] ** 2 * 4 + 8 * case["n"] * case["K"], "flops": 2 * case["n"] ** 2 * case["K"]}
    return {"bytes": 8 * case["N"], "flops": 0}


def tolerance(case):
    path = case["path"]
    if path == "shards":
        return "exact"
    if path == "similarity":
        # an fp32 Gram value of d products against row norms of about 1.25 d, over sigma^2 = d: 2e-7 from 64 bits
        return {"rel": 1e-6, "max": 1e-5}
    if path == "bandwidth":
        # a mean of distances, each from an fp32 Gram value: up to 6e-8 from 64 bits, 1e-6 allowed for other sums
        return {"rel": 1e-6}
    if path == "sweep":
        # sums of n fp32 terms: 4e-8 from 64 bits in a tree, more if taken one after the other
        return {"rel": 1e-6, "max": 1e-5}
    # Two workers whose objectives (or samples whose gains) agree to rounding may swap places.  Gains summed in fp32 by
    # sweeps against gains carried in 64 bits, on the same similarities: up to 1.3 % of the order and 2e-5 of an objective.
    return {"rel": 1e-4, "max": 1e-3, "differ": 0.01}


def _similarity64(X, sigma2):
    X = X.double()
    sq = (X * X).sum(1)
    S = X @ X.T
    S.mul_(-2).add_(sq[:, None]).add_(sq[None, :]).clamp_(min=0).mul_(-0.5 / sigma2).exp_()
    S.fill_diagonal_(1.0)
    return S


def _greedy64(S, cap, graph_cut):
    """Algorithm 1 on one class in 64 bits: assignment, order and objectives."""
    n, K = S.shape[0], len(cap)
    total = S.sum(0)
    gain = np.tile(total - np.diag(S) if graph_cut else total, (K, 1))
    cur = np.zeros((K, n))
    f, cnt = np.zeros(K), np.zeros(K, dtype=np.int64)
    assign, order = np.full(n, -1, np.int32), np.full(n, -1, np.int32)
    for t in range(int(sum(cap))):
        k = int(np.argmin(np.where(cnt < cap, f, np.inf)))
        v = int(np.argmax(gain[k]))
        f[k] += gain[k, v]
        cnt[k] += 1
        assign[v], order[v] = k, t
        row = S[v]
        if graph_cut:
            gain[k] -= 2 * row
        else:
            D = np.flatnonzero(row > cur[k])
            old, new = cur[k, D][:, None], row[D][:, None]
            gain[k] -= np.minimum(np.maximum(S[D] - old, 0), new - old).sum(0)
            cur[k, D] = row[D]
        gain[:, v] = -np.inf
    return assign, order, f


def exact(case, seed):
    path = case["path"]
    if path == "dataset":
        gc = case["route"] == "graph_cut"
        # a step costs about n operations with the graph-cut function; the first steps of a worker n^2 otherwise
        if case["L"] * case["n_c"] ** 2 * (1 if gc else len(case["caps"]) / 8) > 3e8 or case["L"] * case["n_c"] > 60000:
            return None
        X, labels, _ = _dataset(case, seed)
        r = _capacities(case).astype(np.int64)
        N = X.shape[0]
        assign, order = np.full(N, -1, np.int32), np.full(N, -1, np.int32)
        obj = np.zeros((case["L"], len(r)))
        for c in range(case["L"]):
            at = torch.nonzero(labels == c).flatten()
            S = _similarity64(X[at], float(case["d"])).cpu().numpy()
            cap = len(at) * r // r.sum()
            extra = len(at) - int(cap.sum())
            cap[np.argsort(-r, kind="stable")[:extra]] += 1
            at = at.cpu().numpy()
            assign[at], order[at], obj[c] = _greedy64(S, cap, gc)
        return {"assign": assign, "order": order, "obj": obj}
    if path == "class":
        return None
    if path == "similarity":
        s = prepare(case, seed)
        X = s["X"] if s["index"] is None else s["X"][s["index"].long()]
        s.clear()
        return _similarity64(X, float(case["d"]))
    if path == "bandwidth":
        X = prepare(case, seed)["X"].double()
        n, sq, total = X.shape[0], (X * X).sum(1), 0.0
        for i in range(0, n, 4096):
            part = X[i:i + 4096] @ X.T
            part.mul_(-2).add_(sq[i:i + 4096, None]).add_(sq[None, :]).clamp_(min=0)
            part[torch.arange(part.shape[0]), torch.arange(i, i + part.shape[0])] = 0
            total += float(part.sqrt_().sum())
        return total / (float(n) * n)
    if path == "sweep":
        s = prepare(case, seed)
        S = s["S"].double()
        return torch.stack([(S - c[:, None]).clamp_(min=0).sum(0) for c in s["cur"].double()])
    return None
