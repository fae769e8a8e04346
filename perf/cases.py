"""What a user of this library has it do, as cases that can be timed: train steps (full graph and mini-batch), the
training loops around them, neighbour aggregation on its own, the combination of partition gradients and the
construction of partitions.

Every case goes through the package's public calls.  Graphs are R-MAT graphs (a, b, c = 0.57, 0.19, 0.19) with
scrambled ids, the degree skew of the graphs this library is for; features are N(0, 1), labels uniform, weights
N(0, 1 / fan-in).  Everything is made from the seed alone, on the GPU.
"""
from __future__ import annotations

import ctypes
import math

import torch

import paper_2602_01872_amd as g

DEV = "cuda"
SPLIT = 1                  # the seed by which nodes are dealt to partitions where a case builds them

ARCHS = {"sage": g.ARCH_SAGE_MEAN, "gcn": g.ARCH_GCN, "residual": g.ARCH_GCN_RESIDUAL, "gat": g.ARCH_GAT}
ESTIMATORS = {"none": g.EST_NONE, "node": g.EST_NODE_LEVEL, "mindist": g.EST_BATCH_MIN_DIST, "shrinkage": g.EST_SHRINKAGE}
SCALES = {"none": g.SCALE_NONE, "mean": g.SCALE_MEAN, "rsqrt": g.SCALE_RSQRT}


# ------------------------------------------------------------------------------------------------ the cases
def listed():
    return [
        # One iteration of the phase-parallel loop on a small graph (the first configuration): 4 steps of a 2-layer GCN,
        # the reduction and the update.  Partitions of 2,500 nodes: everything is launches and latency.
        {"name": "iteration_small", "kind": "iterate", "arch": "gcn", "nodes": 10_000, "edges": 100_000, "parts": 4,
         "dims": "64-64-8", "estimator": "shrinkage"},
        # One mini-batch step on a large store (the third configuration): isolated sampling, bf16 features.
        {"name": "minibatch_step", "kind": "minibatch", "nodes": 7_000_000, "edges": 100_000_000, "batch": 1024,
         "fanouts": "15-10-5", "dims": "128-256-256-172", "bf16": True, "dropout": 0.0, "estimator": "mindist"},
        # One epoch of the mini-batch loop as the experiments run it: every partition's training nodes once, batches of
        # 1024, dropout, the shrinkage factor; captured steps on several streams.
        {"name": "minibatch_epoch", "kind": "epoch", "nodes": 600_000, "edges": 15_000_000, "parts": 4, "train": 0.04,
         "batch": 1024, "fanouts": "15-10-5", "dims": "100-256-256-47", "dropout": 0.5, "lanes": 4},
        # The full-graph step of a 3-layer GraphSAGE on one partition's share (the second configuration), with the
        # dropout rate of the experiments, and the reduction over 8 partitions: dense products over 3e5 rows.
        {"name": "sage_step", "kind": "step", "arch": "sage", "nodes": 300_000, "edges": 975_000, "missing": 7,
         "dims": "100-256-256-47", "bf16": False, "dropout": 0.5, "masked": False, "weighted": False,
         "estimator": "shrinkage", "parts": 8},
        # The same step where nothing is a multiple of anything: odd widths, a loss mask, weighted neighbours and
        # per-node loss weights.
        {"name": "sage_step_ragged", "kind": "step", "arch": "sage", "nodes": 100_003, "edges": 1_500_007, "missing": 1,
         "dims": "75-130-41", "bf16": False, "dropout": 0.0, "masked": True, "weighted": True, "estimator": "node",
         "parts": 2},
        # The attention model on the same share.
        {"name": "gat_step", "kind": "step", "arch": "gat", "nodes": 300_000, "edges": 975_000, "missing": 7,
         "dims": "100-256-256-47", "bf16": False, "dropout": 0.0, "masked": False, "weighted": False,
         "estimator": "shrinkage", "parts": 8},
        # A deep residual GCN (the fourth configuration at a quarter of its size, so that several fit the card).
        {"name": "residual_step", "kind": "step", "arch": "residual", "nodes": 1_048_576, "edges": 25_000_000, "missing": 0,
         "dims": "128-256-256-256-256-256-256-256-64", "bf16": False, "dropout": 0.0, "masked": False, "weighted": False,
         "estimator": "none", "parts": 1},
        # A dense share of a very large graph that exists as sorted rows (the fifth configuration at half its nodes and a
        # quarter of its edges): bf16 features, and the reduction over 256 partitions.
        {"name": "dense_share_step", "kind": "share", "nodes": 8_388_608, "edges": 1 << 30, "missing": 255, "dims": "64-128-16",
         "parts": 256},
        # Neighbour aggregation on its own, both directions.
        {"name": "spmm_pair", "kind": "spmm", "nodes": 1_048_576, "edges": 25_000_000, "width": 256, "bf16": False,
         "scale": "mean", "self": False},
        # Many large gradients combined and applied: a stream over memory.
        {"name": "combine_large", "kind": "combine", "parts": 64, "params": 1 << 24, "estimator": "mindist"},
        # One partition of eight out of the whole edge list.
        {"name": "partition_hash", "kind": "build", "way": "hash", "nodes": 2_400_000, "edges": 62_000_000, "parts": 8,
         "width": 100},
        # What a switch of sweeping partitions costs a worker: base + swept chunk, and its rows of the features.
        {"name": "partition_switch", "kind": "build", "way": "chunks", "nodes": 2_400_000, "edges": 62_000_000, "parts": 8,
         "width": 100},
    ]


def _log(rng, lo, hi):
    """A whole number between lo and hi, evenly over the logarithm."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _widths(rng, layers, feat, hidden, classes):
    inner = [_log(rng, *hidden) for _ in range(layers - 1)]
    return "-".join(str(d) for d in [_log(rng, *feat), *inner, _log(rng, *classes)])


def _unit(width, edges):
    """Large matrices are kept in rows of whole 16-byte units; small ones come in any width."""
    return width if edges <= 2_000_000 else (width + 3) // 4 * 4


def draw(rng):
    kind = rng.choice(["iterate", "minibatch", "epoch", "step", "step", "step", "share", "spmm", "combine", "build", "build"])
    est = rng.choice(sorted(ESTIMATORS))
    if kind == "iterate":
        nodes = _log(rng, 2_000, 40_000)
        return {"kind": kind, "arch": rng.choice(["sage", "gcn"]), "nodes": nodes, "edges": _log(rng, 4 * nodes, 16 * nodes),
                "parts": rng.randint(2, 8), "dims": _widths(rng, rng.randint(2, 3), (16, 128), (16, 128), (3, 47)), "estimator": est}
    if kind == "minibatch":
        nodes = _log(rng, 100_000, 7_000_000)
        layers = rng.randint(2, 3)
        return {"kind": kind, "nodes": nodes, "edges": min(100_000_000, _log(rng, 6 * nodes, 20 * nodes)), "batch": _log(rng, 64, 1024),
                "fanouts": "-".join(str(rng.randint(3, 15)) for _ in range(layers)),
                "dims": _widths(rng, layers, (32, 160), (32, 256), (5, 172)), "bf16": rng.random() < 0.5,
                "dropout": rng.choice([0.0, 0.5]), "estimator": est}
    if kind == "epoch":
        nodes = _log(rng, 60_000, 600_000)
        return {"kind": kind, "nodes": nodes, "edges": _log(rng, 8 * nodes, 25 * nodes), "parts": rng.randint(2, 4), "train": 0.04,
                "batch": rng.choice([256, 512, 1000, 1024]), "fanouts": "-".join(str(rng.randint(3, 15)) for _ in range(3)),
                "dims": _widths(rng, 3, (32, 128), (64, 256), (5, 64)), "dropout": rng.choice([0.0, 0.5]), "lanes": rng.choice([1, 4])}
    if kind == "step":
        arch = rng.choice(["sage", "sage", "gcn", "residual", "gat"])
        nodes = _log(rng, 3_000, 250_000)
        edges = _log(rng, 3 * nodes, 12 * nodes)
        if arch == "residual":                             # the same hidden width throughout, so that the skips exist
            hidden, layers = _log(rng, 32, 256), rng.randint(3, 8)
            dims = "-".join(str(d) for d in [_unit(_log(rng, 32, 256), edges), *[hidden] * (layers - 1), _log(rng, 5, 64)])
        else:
            feat, rest = _widths(rng, rng.randint(2, 3), (20, 300), (32, 256), (3, 100)).split("-", 1)
            dims = "%d-%s" % (_unit(int(feat), edges), rest)
        return {"kind": kind, "arch": arch, "nodes": nodes, "edges": edges, "missing": rng.choice([0, 1, 7]),
                "dims": dims, "bf16": arch != "residual" and rng.random() < 0.3, "dropout": rng.choice([0.0, 0.0, 0.5]),
                "masked": rng.random() < 0.3, "weighted": arch == "sage" and rng.random() < 0.25, "estimator": est,
                "parts": rng.randint(1, 8)}
    if kind == "share":
        nodes = _log(rng, 1 << 18, 1 << 23)
        return {"kind": kind, "nodes": nodes, "edges": min(1 << 30, _log(rng, 32 * nodes, 256 * nodes)), "missing": rng.choice([15, 255]),
                "dims": "%d-%d-%d" % (8 * _log(rng, 2, 16), _log(rng, 32, 128), _log(rng, 8, 64)), "parts": _log(rng, 16, 256)}
    if kind == "spmm":
        nodes = _log(rng, 10_000, 1 << 20)
        edges = _log(rng, 4 * nodes, 24 * nodes)
        return {"kind": kind, "nodes": nodes, "edges": edges, "width": _unit(_log(rng, 4, 256), edges),
                "bf16": rng.random() < 0.4, "scale": rng.choice(sorted(SCALES)), "self": rng.random() < 0.4}
    if kind == "combine":
        parts = _log(rng, 2, 256)
        return {"kind": kind, "parts": parts, "params": _log(rng, 2_000, (1 << 30) // max(64, parts)), "estimator": est}
    nodes = _log(rng, 20_000, 2_400_000)
    return {"kind": "build", "way": rng.choice(["hash", "chunks", "weighted", "halo", "local", "rows"]), "nodes": nodes,
            "edges": _log(rng, 8 * nodes, 25 * nodes), "parts": rng.randint(2, 16), "width": _log(rng, 8, 128)}


# ------------------------------------------------------------------------------------------------ inputs
def _gen(seed, stream):
    return torch.Generator(device=DEV).manual_seed(1_000_003 * int(seed) + stream)


def _rmat(nodes, edges, seed):
    """(src, dst), int64: an R-MAT edge list over `nodes` nodes, ids scrambled so that hubs are spread over the range."""
    scale = max(1, (nodes - 1).bit_length())
    mask, half = (1 << scale) - 1, max(1, scale // 2)
    gen = _gen(seed, 1)
    out = torch.empty(2, edges, dtype=torch.int64, device=DEV)
    for lo in range(0, edges, 1 << 26):
        m = min(edges, lo + (1 << 26)) - lo
        s = torch.zeros(m, dtype=torch.int32, device=DEV)
        d = torch.zeros(m, dtype=torch.int32, device=DEV)
        r = torch.empty(m, device=DEV)
        for _ in range(scale):
            r.uniform_(generator=gen)
            low = r >= 0.76                                  # the two quadrants with the source bit set
            s.mul_(2).add_(low)
            d.mul_(2).add_(((r >= 0.57) ^ low) | (r >= 0.95))
        for k, v in enumerate((s, d)):
            x = v.to(torch.int64)
            for odd in (0x9E3779B1, 0x85EBCA77):
                x.mul_(odd).bitwise_and_(mask)
                x.bitwise_xor_(x >> half)
            out[k, lo:lo + m] = x.remainder_(nodes)
    return out[0], out[1]


def _rows(src, dst, nodes):
    """The edge list as rows of in-edges: rowptr int64, col int32, sources ascending in every row."""
    key = torch.sort((dst << 32) | src)[0]
    rowptr = torch.zeros(nodes + 1, dtype=torch.int64, device=DEV)
    torch.cumsum(torch.bincount(dst, minlength=nodes), 0, out=rowptr[1:])
    return rowptr, key.to(torch.int32)


def _global_degree(d_local, missing, seed):
    """In-degrees in the whole graph of nodes that miss about `missing` times their local in-edges."""
    extra = torch.rand(d_local.numel(), generator=_gen(seed, 2), device=DEV) * (2 * missing + 1) * d_local.clamp(min=1)
    return d_local + (extra.to(torch.int64) if missing else 0)


def _relabel(nodes, parts, seed):
    """A random renaming of the nodes that keeps everybody in its partition of the split SPLIT, so that graphs of different
    seeds have partitions of the same size."""
    owner = torch.empty(nodes, dtype=torch.int32, device=DEV)
    g.grp_node_owners(nodes, parts, SPLIT, owner)
    noise = torch.rand(nodes, generator=_gen(seed, 11), device=DEV, dtype=torch.float64)
    name = torch.empty(nodes, dtype=torch.int64, device=DEV)
    name[torch.argsort(owner, stable=True)] = torch.argsort(owner + noise)
    return name


def _features(n, width, bf16, seed):
    return torch.randn(n, width, generator=_gen(seed, 3), device=DEV, dtype=torch.bfloat16 if bf16 else torch.float32)


def _labels(n, classes, seed):
    return torch.randint(classes, (n,), generator=_gen(seed, 4), device=DEV, dtype=torch.int32)


def _mask(n, share, seed):
    return (torch.rand(n, generator=_gen(seed, 5), device=DEV) < share).to(torch.uint8)


def _theta(arch, dims, seed):
    gen, parts = _gen(seed, 6), []
    for fin, fout in zip(dims, dims[1:]):
        for _ in range(2 if arch == "sage" else 1):
            parts.append(torch.randn(fin * fout, generator=gen, device=DEV) * fin ** -0.5)
        if arch == "gat":
            parts.append(torch.randn(2 * fout, generator=gen, device=DEV) * fout ** -0.5)
        parts.append(torch.randn(fout, generator=gen, device=DEV) * 0.1)
    return torch.cat(parts).contiguous()


def _dims(case):
    return [int(d) for d in case["dims"].split("-")]


def _records(stats):
    """The statistics records as numbers: loss, sum of ratios, R; |S|, edges used."""
    return {"real": stats.view(torch.float64).view(-1, 5)[:, :3], "whole": stats.view(torch.int64).view(-1, 5)[:, 3:]}


def _other_parts(parts, ld, seed):
    """Gradients and statistics of `parts` partitions, resident as the reduction finds them (the caller's own step
    overwrites slot 0)."""
    grads = torch.randn(parts, ld, generator=_gen(seed, 7), device=DEV)
    stats = g.new_stats(parts, device=DEV)
    u = torch.rand(parts, generator=_gen(seed, 8), device=DEV, dtype=torch.float64)
    real, whole = stats.view(torch.float64).view(-1, 5), stats.view(torch.int64).view(-1, 5)
    whole[:, 3] = 10_000
    real[:, 1] = 10_000 * (0.2 + 0.5 * u)
    real[:, 2] = torch.floor(1e5 * (0.5 + u))
    return grads, stats


class _Borrowed:
    """One of a partition's device arrays, for torch: a view into the handle, which it keeps alive."""

    def __init__(self, part, ptr, count, typestr):
        self.part = part
        self.__cuda_array_interface__ = {"shape": (count,), "typestr": typestr, "data": (ptr, False), "version": 2}


def _arrays(part):
    n, nnz, v = part.n, part.nnz, part.view
    spec = {"l2g": (n, "<i8"), "rowptr": (n + 1, "<i8"), "col": (nnz, "<i4"), "colptr": (n + 1, "<i8"), "row": (nnz, "<i4"),
            "d_local_in": (n, "<i4"), "d_local_out": (n, "<i4"), "d_global_in": (n, "<i8")}
    return {k: torch.as_tensor(_Borrowed(part, getattr(v, k), c, t), device=DEV) for k, (c, t) in spec.items() if c}


# ------------------------------------------------------------------------------------------------ prepare
def prepare(case, seed):
    return {"iterate": _prepare_iterate, "minibatch": _prepare_minibatch, "epoch": _prepare_epoch, "step": _prepare_step,
            "share": _prepare_step, "spmm": _prepare_spmm, "combine": _prepare_combine, "build": _prepare_build}[case["kind"]](case, seed)


def _hash_parts(case, seed, width):
    """All partitions of a graph with their rows of the features and labels."""
    src, dst = _rmat(case["nodes"], case["edges"], seed)
    parts = [g.grp_partition(src, dst, case["nodes"], case["parts"], seed, p) for p in range(case["parts"])]
    x, y = _features(case["nodes"], width, False, seed), _labels(case["nodes"], _dims(case)[-1], seed)
    l2g = [_arrays(p)["l2g"] for p in parts]
    return parts, [g.grp_gather_rows(x, i) for i in l2g], [g.grp_gather_rows(y, i) for i in l2g], l2g


def _prepare_iterate(case, seed):
    dims = _dims(case)
    parts, xs, ys, _ = _hash_parts(case, seed, dims[0])
    trainer = g.PhaseParallelTrainer(parts, g.model_desc(ARCHS[case["arch"]], dims), xs, ys, [None] * len(parts),
                                     _theta(case["arch"], dims, seed), ESTIMATORS[case["estimator"]], len(parts))
    return {"run": _run_trainer, "trainer": trainer}


def _prepare_epoch(case, seed):
    dims = _dims(case)
    parts, xs, ys, l2g = _hash_parts(case, seed, dims[0])
    train = _mask(case["nodes"], case["train"], seed)
    masks = [g.grp_gather_rows(train, i) for i in l2g]
    trainer = g.MiniBatchTrainer(parts, g.model_desc(g.ARCH_SAGE_MEAN, dims), xs, ys, masks, _theta("sage", dims, seed),
                                 g.EST_SHRINKAGE, len(parts), case["batch"], [int(f) for f in case["fanouts"].split("-")], seed,
                                 g.optimizer_desc(g.OPT_SGD, lr=0.003), dropout_rate=case["dropout"], dropout_seed=seed,
                                 lanes=case["lanes"], graphs=True)
    return {"run": _run_trainer, "trainer": trainer}


def _run_trainer(s):
    t = s["trainer"]
    t.run_epoch()
    return {"theta": t.theta, "m": t.m, "v": t.v, "update": t.update, "grads": t.grads, "stats": _records(t.stats)}


def _prepare_minibatch(case, seed):
    dims, n = _dims(case), case["nodes"]
    src, dst = _rmat(n, case["edges"], seed)
    d_global = _global_degree(torch.bincount(dst, minlength=n), 15, seed)
    part = g.grp_partition_from_local_coo(src, dst, n, d_global_in=d_global)
    del src, dst
    seeds = torch.randperm(n, generator=_gen(seed, 9), device=DEV)[:case["batch"]].to(torch.int32)
    opts = g.step_opts(estimator=ESTIMATORS[case["estimator"]], full_graph=False, seeds=seeds,
                       fanouts=[int(f) for f in case["fanouts"].split("-")], sampler_seed=seed, batch_id=0,
                       dropout_rate=case["dropout"], dropout_seed=seed)
    model = g.model_desc(g.ARCH_SAGE_MEAN, dims, feat_dtype=g.DTYPE_BF16 if case["bf16"] else g.DTYPE_FP32)
    return _step_state(part, model, opts, "sage", dims, case["bf16"], None, 1, seed)


def _prepare_step(case, seed):
    dims, n, share = _dims(case), case["nodes"], case["kind"] == "share"
    arch, bf16 = ("sage", True) if share else (case["arch"], case["bf16"])
    if not share and case["weighted"]:                       # half of a graph of twice the nodes
        src, dst = _rmat(2 * n, 4 * case["edges"], seed)
        w = torch.exp(torch.rand(src.numel(), generator=_gen(seed, 10), device=DEV) * 2.772588 - 1.386294)   # in [1/4, 4)
        part = g.grp_partition_weighted(src, dst, w, 2 * n, 2, seed, 0)
    else:
        src, dst = _rmat(n, case["edges"], seed)
        d_global = _global_degree(torch.bincount(dst, minlength=n), case["missing"], seed)
        if share:
            rowptr, col = _rows(src, dst, n)
            del src, dst
            part = g.grp_partition_from_csr(rowptr, col, n, d_global_in=d_global)
        else:
            part = g.grp_partition_from_local_coo(src, dst, n, d_global_in=d_global)
            del src, dst
    opts = g.step_opts(estimator=g.EST_SHRINKAGE if share else ESTIMATORS[case["estimator"]], full_graph=True,
                       dropout_rate=0.0 if share else case["dropout"], dropout_seed=seed)
    model = g.model_desc(ARCHS[arch], dims, feat_dtype=g.DTYPE_BF16 if bf16 else g.DTYPE_FP32)
    mask = _mask(part.n, 0.6, seed) if not share and case["masked"] else None
    return _step_state(part, model, opts, arch, dims, bf16, mask, case["parts"], seed)


def _step_state(part, model, opts, arch, dims, bf16, mask, parts, seed):
    P = g.grp_param_count(model)
    ld = (P + 3) // 4 * 4
    grads, stats = _other_parts(parts, ld, seed)
    return {"run": _run_step, "part": part, "model": model, "opts": opts, "x": _features(part.n, dims[0], bf16, seed),
            "y": _labels(part.n, dims[-1], seed), "mask": mask, "theta": _theta(arch, dims, seed), "P": P, "ld": ld,
            "grads": grads, "stats": stats, "own": stats[:g.STATS_BYTES], "parts": parts,
            "ws": torch.empty(g.grp_step_workspace_bytes(part, model, opts), dtype=torch.uint8, device=DEV),
            "update": torch.zeros(P, device=DEV)}


def _run_step(s):
    g.grp_train_step(s["part"], s["model"], s["opts"], s["x"], s["y"], s["mask"], s["theta"], s["ws"], s["grads"][0], s["own"])
    if s["parts"] > 1:
        g.grp_aggregate(s["grads"], s["ld"], s["stats"], s["parts"], s["P"], s["opts"].estimator, s["update"])
    return {"grad": s["grads"][0], "update": s["update"], "stats": _records(s["own"])}


def _prepare_spmm(case, seed):
    n, F = case["nodes"], case["width"]
    src, dst = _rmat(n, case["edges"], seed)
    part = g.grp_partition_from_local_coo(src, dst, n)
    return {"run": _run_spmm, "part": part, "x": _features(n, F, case["bf16"], seed), "F": F, "scale": SCALES[case["scale"]],
            "self": case["self"], "dtype": g.DTYPE_BF16 if case["bf16"] else g.DTYPE_FP32,
            "y": torch.empty(n, F, device=DEV), "yt": torch.empty(n, F, device=DEV)}


def _run_spmm(s):
    F = s["F"]
    g.grp_spmm(s["part"], False, s["scale"], s["self"], F, s["x"], F, s["dtype"], s["y"], F)
    g.grp_spmm(s["part"], True, s["scale"], s["self"], F, s["x"], F, s["dtype"], s["yt"], F)
    return [s["y"], s["yt"]]


def _prepare_combine(case, seed):
    P = case["params"]
    ld = (P + 3) // 4 * 4
    grads, stats = _other_parts(case["parts"], ld, seed)
    return {"run": _run_combine, "grads": grads, "stats": stats, "parts": case["parts"], "P": P, "ld": ld,
            "variant": ESTIMATORS[case["estimator"]], "update": torch.empty(P, device=DEV), "c": torch.empty(case["parts"], device=DEV),
            "theta": torch.randn(P, generator=_gen(seed, 6), device=DEV), "m": torch.zeros(P, device=DEV),
            "v": torch.zeros(P, device=DEV), "opt": g.optimizer_desc(), "step": 0}


def _run_combine(s):
    s["step"] += 1
    g.grp_aggregate(s["grads"], s["ld"], s["stats"], s["parts"], s["P"], s["variant"], s["update"], s["c"])
    g.grp_optimizer_step(s["opt"], s["P"], s["step"], s["theta"], s["update"], s["m"], s["v"])
    return {"update": s["update"], "c": s["c"], "theta": s["theta"], "m": s["m"], "v": s["v"]}


def _prepare_build(case, seed):
    N, way = case["nodes"], case["way"]
    src, dst = _rmat(N, case["edges"], 1)
    name = _relabel(N, case["parts"], seed)
    src, dst = name[src], name[dst]
    s = {"run": _run_build, "way": way, "N": N, "parts": case["parts"], "x": None}
    if way == "chunks":
        s.update(chunks=g.grp_chunks_build(src, dst, N, case["parts"], SPLIT), x=_features(N, case["width"], False, seed))
    elif way == "rows":
        rowptr, col = _rows(src, dst, N)
        s.update(rowptr=rowptr, col=col, degree=_global_degree(rowptr[1:] - rowptr[:-1], 3, seed))
    else:
        s.update(src=src, dst=dst)
        if way == "weighted":
            s["w"] = torch.rand(src.numel(), generator=_gen(seed, 10), device=DEV) + 0.25
    return s


def _run_build(s):
    way, N, K = s["way"], s["N"], s["parts"]
    if way == "hash":
        part = g.grp_partition(s["src"], s["dst"], N, K, SPLIT, 0)
    elif way == "chunks":
        part = g.grp_partition_from_chunks(s["chunks"], 0, 1)
    elif way == "weighted":
        part = g.grp_partition_weighted(s["src"], s["dst"], s["w"], N, K, SPLIT, 0)
    elif way == "halo":
        part = g.grp_partition_halo(s["src"], s["dst"], N, K, SPLIT, 0, 1)
    elif way == "local":
        part = g.grp_partition_from_local_coo(s["src"], s["dst"], N)
    else:
        part = g.grp_partition_from_csr(s["rowptr"], s["col"], N, d_global_in=s["degree"])
    out = _arrays(part)
    if way == "weighted":
        w = g.PartitionWeights()
        if g.load().grp_partition_weights(part.handle, ctypes.byref(w)) != g.OK:
            raise RuntimeError("grp_partition_weights failed")
        for k, count, t in (("csr_w", part.nnz, "<f4"), ("csc_w", part.nnz, "<f4"), ("w_local_in", part.n, "<f8"),
                            ("w_global_in", part.n, "<f8")):
            out[k] = torch.as_tensor(_Borrowed(part, getattr(w, k), count, t), device=DEV)
    if s["x"] is not None:
        out["x"] = g.grp_gather_rows(s["x"], out["l2g"])
    return out


def run(state):
    return state["run"](state)


# ------------------------------------------------------------------------------------------------ work
def _step_work(arch, dims, n, edges, elem, structure=True):
    """One train step over n nodes and `edges` edges: features, labels, structure (both directions), weights and gradient
    once; one aggregation forward at the narrower width and one back (none below the first layer), the dense products
    of both directions."""
    mats = 2 if arch == "sage" else 1
    params = sum(mats * a * b + b for a, b in zip(dims, dims[1:]))
    flops = 0.0
    for l, (a, b) in enumerate(zip(dims, dims[1:])):
        width = min(a, b) if arch == "sage" else b
        flops += 2.0 * edges * width * (2 if l > 0 or arch != "sage" else 1) * (2 if arch == "gat" else 1)
        flops += 2.0 * n * a * b * mats * (3 if l > 0 else 2)
    structure_bytes = 2.0 * (4.0 * edges + 8.0 * (n + 1)) if structure else 4.0 * edges
    return elem * n * dims[0] + 4.0 * n + structure_bytes + 8.0 * params, flops


def _sampled_work(case, n, mean_degree, batch, elem):
    """One mini-batch step: the blocks a graph of this mean degree gives on average."""
    dims, fanouts = _dims(case), [int(f) for f in case["fanouts"].split("-")]
    rows, total, flops, params = float(batch), 0.0, 0.0, 0
    for l in range(len(fanouts) - 1, -1, -1):
        a, b = dims[l], dims[l + 1]
        edges = rows * min(float(fanouts[l]), mean_degree)
        params += 2 * a * b + b
        flops += 2.0 * rows * a * b * 2 * (3 if l > 0 else 2) + 2.0 * edges * min(a, b) * (2 if l > 0 else 1)
        total += 4.0 * edges
        src = min(float(n), rows + edges)
        if l == 0:
            total += elem * src * a
        rows = src
    return total + 8.0 * params, flops


def work(case):
    kind = case["kind"]
    if kind == "iterate":
        dims = _dims(case)
        b, f = _step_work(case["arch"], dims, case["nodes"], case["edges"] / case["parts"], 4)
        return {"bytes": b, "flops": f}
    if kind == "minibatch":
        b, f = _sampled_work(case, case["nodes"], case["edges"] / case["nodes"], case["batch"], 2 if case["bf16"] else 4)
        return {"bytes": b, "flops": f}
    if kind == "epoch":
        n = case["nodes"] / case["parts"]
        steps = case["parts"] * math.ceil(n * case["train"] / case["batch"])
        batch = n * case["parts"] * case["train"] / steps
        b, f = _sampled_work(case, n, case["edges"] / case["nodes"] / case["parts"], batch, 4)
        return {"bytes": steps * b, "flops": steps * f}
    if kind in ("step", "share"):
        share = kind == "share"
        b, f = _step_work("sage" if share else case["arch"], _dims(case), case["nodes"], case["edges"],
                          2 if share or case["bf16"] else 4)
        return {"bytes": b, "flops": f}
    if kind == "spmm":
        n, e, F = case["nodes"], case["edges"], case["width"]
        return {"bytes": 2.0 * (4.0 * e + 8.0 * (n + 1) + (2 if case["bf16"] else 4) * n * F + 4.0 * n * F), "flops": 4.0 * e * F}
    if kind == "combine":
        P, K = case["params"], case["parts"]
        return {"bytes": 4.0 * P * (K + 1) + 28.0 * P, "flops": 2.0 * P * K + 12.0 * P}
    N, E, K = case["nodes"], case["edges"], case["parts"]
    if case["way"] in ("local", "rows"):
        n, e, read = N, E, 16.0 * E if case["way"] == "local" else 4.0 * E + 8.0 * (N + 1)
    elif case["way"] == "chunks":
        n, e = 2 * N / K, 4 * E / K ** 2
        read = 16.0 * e + 8.0 * n
    else:
        n, e, read = N / K, E / K ** 2, (20.0 if case["way"] == "weighted" else 16.0) * E
        if case["way"] == "halo":
            n, e = n + min(N - n, E / K), E / K
    rows = 8.0 * n * case["width"] if case["way"] == "chunks" else 0.0
    return {"bytes": read + 8.0 * e + 40.0 * n + rows, "flops": 0.0}


# ------------------------------------------------------------------------------------------------ tolerance
def tolerance(case):
    kind = case["kind"]
    if kind == "build":
        return "exact"
    if kind in ("spmm", "combine"):
        return {"rel": 1e-5, "max": 1e-4}
    # A train step is sums in fp32, good to about 1e-6; but the derivative of ReLU takes a decision at every hidden unit of
    # every node, and a pre-activation within rounding of zero (a share of about 1e-7 of them) decides differently after
    # another order of summation.  One such decision moves the gradient of a batch of 1024 seeds by up to 3e-4 of its
    # norm (found by moving the weights by 6e-8 of their size), that of a whole partition by 1e-5.
    return {"rel": 5e-4, "max": 0.1}
