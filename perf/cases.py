"""The workloads whose speed this framework is judged by: trees and forests over record
matrices resident on the GPU, and one over records in host memory.

A case names a tree (or a forest of trees of one shape), a record matrix and the call: the
decomposition, the record type and the kind of result.  Trees and records are synthetic and
made from the seed.  The path-array decomposition is left out: it is kept for comparison
with the paper's mechanism and nobody classifies with it in earnest.
"""
import math

import numpy as np
import torch

from paper_1111_1373_amd import dtree as dt
from paper_1111_1373_amd import workloads as W

TORCH_TYPES = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16,
               "u8": torch.uint8}
ELEM_BYTES = {"f32": 4, "f16": 2, "bf16": 2, "u8": 1}


def _case(name, kind, shape, size, n, features, classes, **more):
    """shape/size: "complete" of depth `size`, "grown" to depth <= `size` (at most 1,023
    decision nodes), "random" with `size` decision nodes, "paper" (15 nodes, depth 11).
    pad: columns of the table beyond those the tree reads."""
    c = {"name": name, "kind": kind, "shape": shape, "size": size, "n": n,
         "features": features, "classes": classes, "trees": 1, "type": "f32",
         "dist": "uniform", "pad": 0, "algo": "data", "out": "class_u8"}
    c.update(more)
    return c


def listed():
    return [
        # A 256 x 256 image of 8 attributes under a small tree: the smallest configuration;
        # the launch and its latency are all there is.
        _case("small_image", "tree", "complete", 4, 65_536, 8, 4),
        # The paper's own experiment: 65,536 records of 19 attributes, a 31-node tree, the
        # speculative decomposition.
        _case("paper_image", "tree", "paper", 11, 65_536, 19, 7, algo="speculative"),
        # One HD video frame, 32 attributes a pixel, an unbalanced tree.
        _case("hd_frame", "tree", "grown", 16, 2_073_600, 32, 16, dist="normal"),
        # The bandwidth-bound batch, the framework's headline benchmark.
        _case("batch", "tree", "complete", 12, 16_777_216, 64, 32),
        # The same batch as 8-bit records (quantised attributes).
        _case("batch_u8", "tree", "complete", 12, 16_777_216, 64, 32, type="u8"),
        # A table of 19 attributes in an odd number of rows, leaf numbers out (they index
        # per-leaf statistics): row widths follow the data set, not the hardware.
        _case("odd_table", "tree", "random", 300, 3_000_001, 19, 11, out="leaf_i32"),
        # The attribute columns of a wider table (label and id columns beside them) read in
        # place through the row stride.
        _case("column_slice", "tree", "random", 1023, 500_001, 100, 9, pad=5,
              algo="speculative", out="class_i32"),
        # Wide rows in half precision (descriptor vectors), speculative decomposition.
        _case("wide_f16", "tree", "complete", 10, 1_000_003, 200, 10, type="f16",
              algo="speculative"),
        # A tree grown to purity: its tables exceed what a compute unit holds on chip.
        _case("large_tree", "tree", "random", 20_000, 1_000_000, 16, 32, out="class_i32"),
        # The random-forest extension: 32 complete trees over 4 million records.
        _case("forest", "forest", "complete", 10, 4_194_304, 32, 8, trees=32),
        # A forest of irregular trees, as training leaves them, on rows of 19 attributes.
        _case("forest_odd", "forest", "random", 255, 300_001, 19, 7, trees=100,
              out="class_i32"),
        # Records in host memory, pageable, classified through the copy pipeline (the
        # paper's outer time).
        _case("host_records", "host", "complete", 8, 1_000_000, 32, 8),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choices(["tree", "forest", "host"], [6, 3, 1])[0]
    features = rng.choice([_log_int(rng, 2, 256), rng.choice([8, 16, 19, 20, 32, 64, 100, 128])])
    pad = rng.choice([0, 0, 0, rng.randint(1, 8)])
    dist = rng.choice(["uniform", "uniform", "normal"])
    algo = rng.choice(["data", "data", "speculative"])
    if kind == "forest":
        x_type, classes = "f32", rng.randint(2, 64)
        trees = _log_int(rng, 4, 128)
        shape = rng.choice(["complete", "grown", "random"])
        size = {"complete": rng.randint(4, 10), "grown": rng.randint(6, 16),
                "random": _log_int(rng, 15, 1023)}[shape]
        steps = trees * (size if shape == "complete" else 16)
        n = min(_log_int(rng, 1000, 4_000_000), 100_000_000 // steps, (1 << 27) // (features + pad))
        out = rng.choice(["class_u8", "class_i32"])
        if algo == "speculative":
            n = max(1000, n // 4)
    else:
        x_type = rng.choices(["f32", "f16", "bf16", "u8"], [5, 2, 2, 2])[0]
        classes, trees = rng.randint(2, 256), 1
        shape = rng.choice(["complete", "grown", "random", "paper"])
        size = {"complete": rng.randint(2, 14), "grown": rng.randint(6, 16),
                "random": _log_int(rng, 15, 20_000), "paper": 11}[shape]
        n = min(_log_int(rng, 1000, 8_000_000), (1 << 27) // (features + pad))
        if kind == "host":
            n = min(n, (1 << 25) // (features + pad))
        out = rng.choice(["class_u8", "class_i32", "leaf_i32"])
    c = _case("", kind, shape, size, n, features, classes, trees=trees, type=x_type,
              dist=dist, pad=pad, algo=algo, out=out)
    del c["name"]
    return c


def _one_tree(c, rng):
    F, C, dist = c["features"], c["classes"], c["dist"]
    if c["shape"] == "complete":
        return W.complete_tree(rng, c["size"], F, C, dist)
    if c["shape"] == "grown":
        return W.grown_tree(rng, 0.85, c["size"], 1023, F, C, dist)
    if c["shape"] == "random":
        pool = W.normal_f32(rng, 4096) if dist == "normal" else None
        return W.random_full_tree(rng, c["size"], F, C, threshold_values=pool)
    return W.paper_shape_tree(rng, 15, c["size"], F, C, spine_p=0.8)


def _trees(c, seed):
    rng = np.random.Generator(np.random.PCG64(np.random.SeedSequence([seed, 1])))
    trees = [W.narrow_tree(_one_tree(c, rng), c["type"], c["dist"]) for _ in range(c["trees"])]
    off = np.zeros(len(trees) + 1, dtype=np.int32)
    off[1:] = np.cumsum([len(t) for t in trees])
    return np.concatenate(trees), off


def _records(c, seed):
    """The record matrix on the GPU: columns [0, features) of a table `pad` columns wider."""
    n, ld = c["n"], c["features"] + c["pad"]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    table = torch.empty((n, ld), dtype=TORCH_TYPES[c["type"]], device="cuda")
    draw_block = torch.randn if c["dist"] == "normal" else torch.rand
    rows = max(1, (1 << 28) // ld)
    for r in range(0, n, rows):
        x = draw_block((min(rows, n - r), ld), device="cuda", generator=gen)
        if c["type"] == "u8":      # the quantisation that narrow_tree() gives the thresholds
            x = x.mul_(32).add_(128) if c["dist"] == "normal" else x.mul_(256)
            x = x.floor_().clamp_(0, 255)
        table[r:r + rows] = x
    return table[:, :c["features"]]


def prepare(case, seed):
    nodes, off = _trees(case, seed)
    F, C = case["features"], case["classes"]
    x = _records(case, seed)
    s = {"algo": case["algo"], "out": case["out"], "x": x}
    if case["kind"] == "forest":
        s["model"] = dt.Forest(nodes, off, F, C)
    else:
        s["model"] = dt.Tree(nodes, F, C)
    if case["kind"] == "host":
        x = x.cpu()
        bits = case["type"] == "bf16"
        s["x"] = (x.view(torch.int16).numpy().view(np.uint16) if bits else x.numpy())
        s["x_type"] = case["type"]
        s["pipeline"] = dt.Pipeline(F)
    return s


def run(state):
    if "pipeline" in state:
        return state["pipeline"].classify(state["model"], state["x"], algo=state["algo"],
                                          out_kind=state["out"], x_type=state["x_type"])
    return state["model"].classify(state["x"], algo=state["algo"], out_kind=state["out"])


def _steps(case):
    """Comparisons a record makes in one tree of about this shape."""
    if case["shape"] in ("complete", "paper"):
        return case["size"]
    if case["shape"] == "grown":
        return min(case["size"], 10)
    return max(1.0, 1.4 * math.log2(case["size"] + 1))


def work(case):
    out_bytes = 1 if case["out"] == "class_u8" else 4
    row = case["features"] * ELEM_BYTES[case["type"]]
    return {"bytes": case["n"] * (row + out_bytes),
            "flops": case["n"] * case["trees"] * _steps(case)}


def tolerance(case):
    return "exact"      # labels and leaf numbers, decided by exact comparisons


def exact(case, seed):
    """Every record walked node by node with the stored values widened to 64 bits."""
    nodes, off = _trees(case, seed)
    x = _records(case, seed)
    dev = x.device
    feature = torch.from_numpy(nodes["feature"].astype(np.int64)).to(dev)
    threshold = torch.from_numpy(nodes["threshold"].astype(np.float64)).to(dev)
    left = torch.from_numpy(nodes["left"].astype(np.int64)).to(dev)
    cls = torch.from_numpy(nodes["cls"].astype(np.int64)).to(dev)
    got = torch.empty(case["n"], dtype=torch.uint8 if case["out"] == "class_u8" else torch.int32,
                      device=dev)
    C, step = case["classes"], 1 << 21
    for r in range(0, case["n"], step):
        block = x[r:r + step]
        rows = torch.arange(block.shape[0], device=dev)
        votes = torch.zeros((block.shape[0], C), dtype=torch.int64, device=dev)
        for k in range(case["trees"]):
            at = torch.full_like(rows, int(off[k]))
            while True:
                inner = cls[at] < 0
                if not bool(inner.any()):
                    break
                right = ~(block[rows, feature[at]].double() < threshold[at])
                at = torch.where(inner, int(off[k]) + left[at] + right, at)
            if case["kind"] == "forest":
                votes[rows, cls[at]] += 1
        if case["kind"] == "forest":   # most votes, the smallest class among equals
            value = (votes * C + torch.arange(C - 1, -1, -1, device=dev)).argmax(1)
        else:
            value = at if case["out"] == "leaf_i32" else cls[at]
        got[r:r + step] = value.to(got.dtype)
    return got.cpu().numpy() if case["kind"] == "host" else got
