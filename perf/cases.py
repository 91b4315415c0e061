"""The work that a user of the random-forest performance model has it do.

A case names one pass through the public binding (paper_1811_00156_amd.rf):
binning a feature frame, fitting a forest, a tuning grid or a leave-one-out
study, predicting, choosing a device, serving a request stream and saving a
forest.  Frames are the synthetic stand-ins of paper_1811_00156_amd.synth
(n_vec feature vectors replicated over n_dev devices, p features), cut to n
rows where a case asks for a ragged size; the forest seed is the inputs' seed.

Keys every case has: kind, n_vec, n_dev, p, n (rows of the frame), bins.
Forest cases add trees, mtry, min_node and bootstrap; the others are described
at their kind.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1811_00156_amd import rf, synth

# The paper's frame: 37 kernels x 4 sizes on 15 devices, 34 features.
_SMALL = {"n_vec": 148, "n_dev": 15, "p": 34, "n": 2220}
# The large frame of the benchmark: 6250 vectors on 32 devices, 64 features.
_LARGE = {"n_vec": 6250, "n_dev": 32, "p": 64, "n": 200000}
_LARGE_FOREST = {**_LARGE, "bins": 256, "trees": 500, "mtry": 16, "min_node": 5, "bootstrap": True}
_PAPER_FOREST = {**_SMALL, "bins": 256, "trees": 505, "mtry": 30, "min_node": 9, "bootstrap": True}


def listed():
    return [
        # a scheduler asks for one kernel's time on one device: latency and launches
        {"name": "predict_1", "kind": "predict", **_PAPER_FOREST, "rows": 1, "noalloc": False},
        # a scheduler asks which of the 15 devices runs a kernel's four problem sizes fastest
        {"name": "select_4", "kind": "select", **_PAPER_FOREST, "rows": 4},
        # the largest request of the serving stream, on the 200000-row forest
        {"name": "predict_4096", "kind": "predict", **_LARGE_FOREST, "rows": 4096, "noalloc": False},
        # every row of a large frame predicted in one batch
        {"name": "predict_200000", "kind": "predict", **_LARGE_FOREST, "rows": 200000, "noalloc": False},
        # quantile binning of the large frame, thresholds fitted
        {"name": "bin_200000", "kind": "bin", **_LARGE, "bins": 256, "apply": False},
        # the whole hot path once on the paper's frame: bin, fit 100 trees, predict the frame
        {"name": "fit_100x2220", "kind": "fit", **_SMALL, "bins": 64, "trees": 100, "mtry": 6, "min_node": 5,
         "bootstrap": True, "oob": False},
        # a large forest on the paper's frame, lossless bins, with its predictions and out-of-bag error
        {"name": "fit_2000x2220", "kind": "fit", **_SMALL, "bins": 256, "trees": 2000, "mtry": 12, "min_node": 1,
         "bootstrap": True, "oob": True},
        # a forest on the large frame, and its predictions
        {"name": "fit_500x200000", "kind": "fit", **_LARGE_FOREST, "oob": False},
        # the tuning grid: 10 folds x mtry 1..34 x min.node.size 1,3,5,7,9, scored out of bag
        {"name": "grid_1700", "kind": "grid", **_SMALL, "bins": 64, "trees": 256, "folds": 10, "mtry_max": 34,
         "min_nodes": "1,3,5,7,9"},
        # one forest per left-out kernel, scored on the kernel it has not seen
        {"name": "leave_one_out_37", "kind": "study", **_PAPER_FOREST, "groups": 37},
        # a burst of requests of 1 to 4096 rows answered by the server
        {"name": "serve_48", "kind": "serve", **_LARGE_FOREST, "requests": 48, "max_rows": 4096, "streams": 4},
        # a fitted forest's node arrays taken to the host, as for saving it
        {"name": "export_500", "kind": "export", **_SMALL, "bins": 256, "trees": 500, "mtry": 17, "min_node": 5,
         "bootstrap": True},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _frame(rng, n_max):
    """A frame of up to n_max rows; odd sizes cut the last vectors short."""
    n_dev = rng.choice([1, 2, 5, 15, 15, 32])
    n = _log_int(rng, 60, n_max)
    n_vec = max(4, -(-n // n_dev))
    return {"n_vec": n_vec, "n_dev": n_dev, "p": rng.randint(3, 80), "n": min(n, n_vec * n_dev)}


def _forest(rng, f, budget):
    """Forest parameters whose rows x trees x mtry stay within `budget`."""
    mtry = rng.randint(1, f["p"] + 1)
    most = max(1, min(2000, int(budget / (f["n"] * max(mtry, 8)))))
    return {**f, "bins": rng.choice([16, 64, 64, 128, 256, 256, rng.randint(2, 256)]), "trees": _log_int(rng, 1, most),
            "mtry": mtry, "min_node": rng.choice([1, 2, 5, 9, rng.randint(1, 50)]), "bootstrap": rng.random() < 0.9}


def draw(rng):
    kind = rng.choice(["predict", "predict", "select", "bin", "fit", "fit", "fit", "grid", "study", "serve", "export"])
    if kind == "bin":
        f = _frame(rng, 200000)
        return {"kind": kind, **f, "bins": rng.randint(2, 256), "apply": rng.random() < 0.4}
    if kind == "fit":
        return {"kind": kind, **_forest(rng, _frame(rng, 200000), 5e8), "oob": rng.random() < 0.4}
    if kind == "grid":
        n_dev = rng.choice([5, 15])
        n_vec = rng.randint(20, 300)
        p = rng.randint(6, 40)
        return {"kind": kind, "n_vec": n_vec, "n_dev": n_dev, "p": p, "n": n_vec * n_dev - rng.randint(0, 4),
                "bins": rng.choice([32, 64, 256]), "trees": _log_int(rng, 8, 128), "folds": rng.randint(2, 6),
                "mtry_max": rng.randint(1, min(p, 16)), "min_nodes": rng.choice(["5", "1,9", "1,3,5,7,9", "2,50"])}
    if kind == "study":
        groups = rng.randint(4, 40)
        n_dev = rng.choice([5, 15])
        f = {"n_vec": 4 * groups, "n_dev": n_dev, "p": rng.randint(6, 40), "n": 4 * groups * n_dev}
        return {"kind": kind, **_forest(rng, f, 1e7), "groups": groups}
    f = _forest(rng, _frame(rng, 200000), 1e8)
    if kind == "predict":
        return {"kind": kind, **f, "rows": _log_int(rng, 1, 200000), "noalloc": rng.random() < 0.3}
    if kind == "select":
        return {"kind": kind, **f, "rows": _log_int(rng, 1, 1000)}
    if kind == "serve":
        return {"kind": kind, **f, "requests": rng.randint(4, 60), "max_rows": _log_int(rng, 1, 4096),
                "streams": rng.randint(1, 8)}
    return {"kind": kind, **f}


def _data(case, seed):
    p = case["p"]
    p_ln = max(1, round(p * 20 / 34))
    ds = synth.generate(case["n_vec"], 1, case["n_dev"], p_ln, p - p_ln, min(16, p), seed)
    n = case["n"]
    return ds.X[:n], ds.device[:n], ds.y[:n], ds


def _params(case, seed, mtry=None, min_node=None):
    return rf.make_params(case["trees"], mtry or case["mtry"], min_node or case["min_node"],
                          case.get("bootstrap", True), seed)


def prepare(case, seed):
    dev = torch.device("cuda:0")
    X, d, y, ds = _data(case, seed)
    s = {"case": case, "X": torch.from_numpy(np.ascontiguousarray(X)).to(dev),
         "d": torch.from_numpy(np.ascontiguousarray(d)).to(dev),
         "y": torch.from_numpy(np.ascontiguousarray(y)).to(dev), "seed": seed}
    kind = case["kind"]
    rng = np.random.Generator(np.random.PCG64(seed + 1))
    if kind == "bin":
        if case["apply"]:  # thresholds fitted on another frame of the same columns
            Y, e, _, _ = _data(case, seed + 7)
            _, s["binner"] = rf.aiwc_rf_bin(torch.from_numpy(np.ascontiguousarray(Y)).to(dev),
                                            torch.from_numpy(np.ascontiguousarray(e)).to(dev), case["n_dev"],
                                            case["bins"])
        return s
    if kind == "fit":
        s["params"] = _params(case, seed)
        return s
    s["codes"], s["binner"] = rf.aiwc_rf_bin(s["X"], s["d"], case["n_dev"], case["bins"])
    if kind == "grid":
        fold = rng.permutation(case["n"]) % case["folds"]
        forests = synth.grid_forests(case["folds"], case["mtry_max"], [int(v) for v in case["min_nodes"].split(",")])
        s["fold"] = torch.from_numpy(fold.astype(np.int8)).to(dev)
        # training rows of every forest in turn: the frame less its fold
        s["n_train"] = sum(case["n"] - int((fold == f).sum()) for f, _, _ in forests)
        s["heldout"] = np.array([f for f, _, _ in forests], np.int32)
        s["params"] = [_params(case, seed, m, k) for _, m, k in forests]
        return s
    if kind == "study":
        group = (ds.kernel[:case["n"]] // 4).astype(np.int8)
        s["group"] = torch.from_numpy(group).to(dev)
        s["mask"] = synth.leave_one_kernel_out_masks(case["groups"])
        s["params"] = [_params(case, seed)] * case["groups"]
        return s
    s["forest"] = rf.aiwc_rf_fit(s["codes"], s["binner"], s["y"], _params(case, seed))
    if kind == "predict":
        rows = torch.from_numpy(rng.integers(0, case["n"], case["rows"])).to(dev)
        s["query"] = s["codes"][rows].contiguous()
        if case["noalloc"]:
            s["out"] = torch.empty(case["rows"], dtype=torch.float64, device=dev)
    elif kind == "select":
        rows = torch.from_numpy(rng.integers(0, case["n"], case["rows"])).to(dev)
        s["query"] = s["codes"][rows, :case["p"]].contiguous()
    elif kind == "serve":
        host = s["codes"].cpu().numpy()
        # log-uniform sizes, the same for every seed of the inputs
        sizes = np.random.Generator(np.random.PCG64(synth.SEED_REQUESTS))
        size = np.exp(sizes.uniform(0.0, math.log(case["max_rows"] + 1), case["requests"])).astype(np.int64)
        size = np.clip(size, 1, case["max_rows"])
        s["requests"] = [np.ascontiguousarray(host[rng.integers(0, case["n"], int(k))]) for k in size]
        s["answers"] = [np.zeros(int(k), np.float64) for k in size]
        s["server"] = rf.Server(s["forest"], n_streams=case["streams"])
    elif kind == "export":  # arrays that hold the largest forest of these sizes
        cap = case["trees"] * (2 * case["n"] - 1)
        s["out"] = {"size": np.zeros(case["trees"], np.int64), "col": np.zeros(cap, np.uint8),
                    "bin": np.zeros(cap, np.uint8), "left": np.zeros(cap, np.int32), "q": np.zeros(cap, np.int64),
                    "N": np.zeros(cap, np.int32)}
    return s


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "predict":
        if case["noalloc"]:
            return rf.aiwc_rf_predict_noalloc(s["forest"], s["query"], s["out"])
        return rf.aiwc_rf_predict(s["forest"], s["query"])
    if kind == "select":
        best, times = rf.aiwc_rf_select_device(s["forest"], s["query"], n_devices=case["n_dev"])
        return {"best": best, "times": times}
    if kind == "bin":
        codes, binner = rf.aiwc_rf_bin(s["X"], s["d"], case["n_dev"], case["bins"], s.get("binner"))
        n_bins, thresholds = binner.export()
        return {"codes": codes, "n_bins": n_bins, "thresholds": thresholds}
    if kind == "fit":
        codes, binner = rf.aiwc_rf_bin(s["X"], s["d"], case["n_dev"], case["bins"])
        forest = rf.aiwc_rf_fit(codes, binner, s["y"], s["params"])
        out = {"codes": codes, "yhat": rf.aiwc_rf_predict(forest, codes)}
        if case["oob"]:
            r = rf.aiwc_rf_oob_error(forest, codes, s["y"], n_train=case["n"])
            out.update(sums=r.sums, counts=r.counts, mse=r.mse, mae=r.mae, rows=r.rows)
        return out
    if kind == "grid":
        forest = rf.aiwc_rf_fit(s["codes"], s["binner"], s["y"], s["params"], s["fold"], s["heldout"])
        r = rf.aiwc_rf_oob_error(forest, s["codes"], s["y"], n_train=s["n_train"])
        return {"sums": r.sums, "counts": r.counts, "mse": r.mse, "mae": r.mae, "rows": r.rows}
    if kind == "study":
        forest = rf.aiwc_rf_fit_groups(s["codes"], s["binner"], s["y"], s["params"], s["group"], s["mask"])
        r = rf.aiwc_rf_heldout_error(forest, s["codes"], s["y"], n_heldout=case["n"])
        return {"sums": r.sums, "mse": r.mse, "mae": r.mae, "rows": r.rows}
    if kind == "serve":
        for codes, out in zip(s["requests"], s["answers"]):
            s["server"].submit(codes, out)
        s["server"].drain()
        s["server"].poll()
        return s["answers"]
    out, at = s["out"], 0
    for i, t in enumerate(s["forest"].export()):
        k = t["col"].size
        out["size"][i] = k
        for f in ("col", "bin", "left", "q", "N"):
            out[f][at:at + k] = t[f]
        at += k
    return out


def _leaves(case, min_node=None):
    """About how many leaves a tree has: one per distinct in-bag row, or per half min.node.size of weight."""
    n = case["n"]
    return max(1.0, min(0.632 * n, 1.5 * n / ((min_node or case["min_node"]) + 1)))


def work(case):
    """Inputs read once and outputs written once; an operation per comparison or histogram addition."""
    kind, n, C = case["kind"], case["n"], case["p"] + 1
    frame = n * (4.0 * case["p"] + 4) + n * C
    if kind == "bin":
        return {"bytes": frame, "flops": n * case["p"] * 8.0}
    if kind == "grid":
        b, f = float(n * (C + 9)), 0.0
        for k in case["min_nodes"].split(","):
            leaves = _leaves(case, int(k))
            levels = math.log2(2 * leaves)
            trees = case["folds"] * case["mtry_max"] * case["trees"]
            b += trees * 24 * leaves
            f += trees * 0.632 * n * levels * (case["mtry_max"] + 1) / 2
        return {"bytes": b, "flops": f}
    leaves = _leaves(case)
    levels = math.log2(2 * leaves)
    words = 16.0 * leaves * case["trees"]  # one 64-bit word per node
    grow = 0.632 * n * levels * case["trees"] * case["mtry"]
    if kind == "fit":
        return {"bytes": frame + n * (C + 16) + 1.5 * words, "flops": grow + n * case["trees"] * levels}
    if kind == "study":
        return {"bytes": n * (C + 9) + 1.5 * words * case["groups"], "flops": grow * case["groups"]}
    if kind == "export":
        return {"bytes": words + 18.0 * 2 * leaves * case["trees"], "flops": 2 * leaves * case["trees"]}
    rows = case["rows"] if kind == "predict" else case.get("rows", 0) * case["n_dev"]
    if kind == "serve":
        rows = case["requests"] * max(1.0, case["max_rows"] / math.log(case["max_rows"] + 1))
    visits = rows * case["trees"] * levels
    return {"bytes": rows * (C + 8) + min(words, 8 * visits), "flops": visits}


def exact(case, seed):
    """Binning in plain numpy; a forest's numbers take minutes to grow that way."""
    if case["kind"] != "bin":
        return None
    X, d, _, _ = _data(case, seed)
    source = _data(case, seed + 7)[0] if case["apply"] else X
    n, p, bins = source.shape[0], case["p"], case["bins"]
    codes = np.zeros((X.shape[0], p + 1), np.uint8)
    n_bins = np.zeros(p + 1, np.int32)
    thresholds = np.zeros((p, 255), np.float32)
    for j in range(p):
        order = np.sort(source[:, j])
        t = np.unique(order)[:-1]
        if t.size + 1 > bins:
            t = order[[(k * n) // bins - 1 for k in range(1, bins)]]
            t = np.unique(t[t < order[-1]])
        thresholds[j, :t.size] = t
        n_bins[j] = t.size + 1
        codes[:, j] = np.searchsorted(t, X[:, j], side="left")
    codes[:, p] = d
    n_bins[p] = case["n_dev"]
    return {"codes": codes, "n_bins": n_bins, "thresholds": thresholds}
