"""Performance cases: what a program that orders and reorders sparse matrices
calls, over the sizes it meets.

A case is a dict of plain values.  ``prepare`` builds its graphs on the GPU
from a seed (every seed relabels the vertices anew, as the generators of
``paper_1610_08128_amd.inputs`` do; the points of a random geometric graph
and the edges a strip drops belong to the case), ``run`` makes one call of a public entry
point, ``work`` counts the bytes that call cannot do without, and ``exact``
gives the matrix-vector product in 64 bits from plain torch.

The graph kinds are those of the package's generators: 2D 5-point and 3D
7-point grids, long strips with 1% of the edges dropped, and random geometric
graphs of several disjoint patches (mean degree 12, stray vertices included).
"""

import math
import os

import numpy as np
import torch

from paper_1610_08128_amd import apply, rcm

# the launch options the package ships for this GPU
MI355X_TABLE = os.path.join(os.path.dirname(rcm.__file__), "tuning", "mi355x.txt")

STATS = ("bandwidth_before", "profile_before", "bandwidth_after", "profile_after",
         "edges_traversed", "num_components", "pseudo_diameter", "num_bfs", "num_levels")


def listed():
    return [
        # the smallest ordering a batch or a request stream holds: a coarse
        # mesh of 1,024 vertices; launches, copies and host work count
        {"name": "order grid2d 32x32", "op": "order", "kind": "grid2d", "a": 32, "b": 32, "c": 1},
        # the smallest benchmark workload
        {"name": "order grid2d 64x64", "op": "order", "kind": "grid2d", "a": 64, "b": 64, "c": 1},
        # a small irregular matrix: several components, rows of up to 30 entries
        {"name": "order rgg 3000", "op": "order", "kind": "rgg", "a": 3001, "b": 3, "c": 1},
        # an ordinary 2D mesh, odd sides (a mid-size request)
        {"name": "order grid2d 223x227", "op": "order", "kind": "grid2d", "a": 223, "b": 227, "c": 1},
        # an ordinary irregular matrix, about the mean request of the stream
        {"name": "order rgg 100000", "op": "order", "kind": "rgg", "a": 100003, "b": 4, "c": 1},
        # an ordinary 3D mesh; the caller keeps its workspace
        {"name": "order grid3d 60x60x61", "op": "order", "kind": "grid3d", "a": 60, "b": 60, "c": 61,
         "workspace": True},
        # the benchmark's default workload, as it runs it: kept workspace,
        # the shipped tuning table
        {"name": "order grid3d 128^3", "op": "order", "kind": "grid3d", "a": 128, "b": 128, "c": 128,
         "workspace": True, "tuned": True},
        # a long, narrow structure (high pseudo-diameter): about 30,000 levels
        {"name": "order strip 32x31250", "op": "order", "kind": "strip", "a": 32, "b": 31250, "c": 1,
         "workspace": True},
        # the cheaper level order (one sort by level, degree and id at the end)
        {"name": "order level sort 96^3", "op": "order", "kind": "grid3d", "a": 96, "b": 96, "c": 96,
         "workspace": True, "label_mode": 2},
        # many independent graphs in one call: sizes log-uniform in 1,000 to
        # 200,000 vertices, kinds in turn
        {"name": "batch of 96", "op": "batch", "graphs": 96, "lo": 1000, "hi": 200000, "sizes": 4},
        # the reordered matrix B = P A P^T with its values
        {"name": "permute grid3d 128^3", "op": "permute", "kind": "grid3d", "a": 128, "b": 128,
         "c": 128, "values": True},
        # the product of a solver on a reordered (banded) matrix
        {"name": "spmv grid3d 128^3", "op": "spmv", "kind": "grid3d", "a": 128, "b": 128, "c": 128,
         "values": True, "banded": True},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_shape(rng, lo, hi):
    """A graph of about a log-uniform number of vertices in [lo, hi]."""
    kind = rng.choice(["grid2d", "grid3d", "rgg", "strip"])
    n = _log_int(rng, lo, hi)
    if kind == "rgg":
        return {"kind": kind, "a": min(n, 1000000), "b": rng.randint(2, 5), "c": 1}
    if kind == "strip":
        k = rng.randint(8, 64)
        return {"kind": kind, "a": k, "b": max(16, min(n // k, 1000000 // k, 31250)), "c": 1}
    if kind == "grid2d":
        a = max(2, int(round(math.sqrt(n) * rng.uniform(0.7, 1.4))))
        return {"kind": kind, "a": a, "b": max(2, n // a), "c": 1}
    a = max(2, int(round(n ** (1 / 3) * rng.uniform(0.8, 1.25))))
    b = max(2, int(round(n ** (1 / 3) * rng.uniform(0.8, 1.25))))
    return {"kind": kind, "a": a, "b": b, "c": max(2, n // (a * b))}


def draw(rng):
    op = rng.choice(["order"] * 6 + ["batch", "permute", "permute", "spmv", "spmv"])
    if op == "batch":
        lo = _log_int(rng, 500, 5000)
        return {"op": op, "graphs": rng.randint(4, 96), "lo": lo,
                "hi": _log_int(rng, 4 * lo, 200000), "sizes": rng.randint(0, 1 << 20)}
    case = {"op": op, **_draw_shape(rng, 500, 2000000), "shape": rng.randint(0, 1 << 30)}
    if op == "order":
        case["workspace"] = rng.random() < 0.5
        case["label_mode"] = rng.choice([0, 0, 0, 0, 1, 2])
        case["pp_variant"] = rng.choice([0, 0, 0, 1])
        case["reverse_mode"] = rng.choice([0, 0, 0, 1])
        case["check_full"] = rng.random() < 0.15
    else:
        case["values"] = rng.random() < 0.75
        if op == "spmv":
            case["banded"] = rng.random() < 0.75
    return case


# --- graphs, built on the GPU ----------------------------------------------

def _grid_edges(a, b, c, dev):
    idx = torch.arange(a * b * c, device=dev).view(a, b, c)
    u = torch.cat([idx[:-1].reshape(-1), idx[:, :-1].reshape(-1), idx[:, :, :-1].reshape(-1)])
    v = torch.cat([idx[1:].reshape(-1), idx[:, 1:].reshape(-1), idx[:, :, 1:].reshape(-1)])
    return u, v


def _rgg_edges(n, patches, gen, dev):
    """Edges of points closer than r in `patches` unit squares, and the
    points' order along their squares."""
    patches = max(1, min(patches, n))
    r = math.sqrt(12.0 / (math.pi * max(1, n // patches)))
    side = max(1, int(1.0 / r))
    xy = torch.rand((n, 2), generator=gen, device=dev, dtype=torch.float64)
    patch = torch.arange(n, device=dev) * patches // n
    cell = torch.clamp((xy * side).long(), max=side - 1)
    cx, cy = cell[:, 0], cell[:, 1]
    key = (patch * side + cx) * side + cy
    key, by = torch.sort(key)
    xy, patch, cx, cy = xy[by], patch[by], cx[by], cy[by]
    us, vs = [], []
    at = torch.arange(n, device=dev)
    for dx, dy in ((0, 0), (0, 1), (1, -1), (1, 0), (1, 1)):
        ok = (cx + dx < side) & (cy + dy >= 0) & (cy + dy < side)
        want = (patch * side + cx + dx) * side + cy + dy
        first = torch.searchsorted(key, want)
        count = torch.where(ok, torch.searchsorted(key, want, right=True) - first, 0)
        u = torch.repeat_interleave(at, count)
        v = torch.repeat_interleave(first - (torch.cumsum(count, 0) - count), count)
        v = v + torch.arange(u.numel(), device=dev)
        near = ((xy[u] - xy[v]) ** 2).sum(1) < r * r
        if dx == 0 and dy == 0:
            near &= u < v
        us.append(u[near])
        vs.append(v[near])
    return torch.cat(us), torch.cat(vs), patch.double() + xy[:, 0]


def _graph(case, gen, banded=False):
    """(n, rowptr, colidx): randomly relabelled, or numbered level by level
    along the structure (the banded form an ordering gives)."""
    dev = torch.device("cuda", torch.cuda.current_device())
    a, b, c = case["a"], case["b"], case["c"]
    shape = torch.Generator(device=dev)
    shape.manual_seed(case.get("shape", 1000 * a + b))
    if case["kind"] == "rgg":
        n = a
        u, v, along = _rgg_edges(n, b, shape, dev)
    else:
        n = a * b * c
        u, v = _grid_edges(a, b, c, dev)
        if case["kind"] == "strip":
            keep = torch.rand(u.numel(), generator=shape, device=dev) >= 0.01
            u, v = u[keep], v[keep]
        at = torch.arange(n, device=dev)
        along = at // (b * c) + at // c % b + at % c
    if banded:
        label = torch.empty(n, dtype=torch.long, device=dev)
        label[torch.argsort(along, stable=True)] = torch.arange(n, device=dev)
    else:
        label = torch.randperm(n, generator=gen, device=dev)
    u, v = label[u], label[v]
    d = torch.arange(n, device=dev)
    key = torch.sort(torch.cat([u, v, d]) * n + torch.cat([v, u, d])).values
    rows = key // n
    rowptr = torch.zeros(n + 1, dtype=torch.int32, device=dev)
    rowptr[1:] = torch.cumsum(torch.bincount(rows, minlength=n), 0)
    return n, rowptr, (key - rows * n).int()


def _batch_shapes(case):
    rng = np.random.default_rng(case["sizes"])
    out = []
    for g in range(case["graphs"]):
        n = float(math.exp(rng.uniform(math.log(case["lo"]), math.log(case["hi"]))))
        if g % 3 == 0:
            a = max(2, int(round(math.sqrt(n))))
            out.append({"kind": "grid2d", "a": a, "b": max(2, int(round(n / a))), "c": 1})
        elif g % 3 == 1:
            a = max(2, int(round(n ** (1 / 3))))
            out.append({"kind": "grid3d", "a": a, "b": a, "c": max(2, int(round(n / (a * a))))})
        else:
            out.append({"kind": "rgg", "a": int(n), "b": int(rng.integers(2, 6)), "c": 1})
    return out


def _normal(count, gen):
    dev = torch.device("cuda", torch.cuda.current_device())
    return torch.randn(count, generator=gen, device=dev, dtype=torch.float64)


def prepare(case, seed):
    dev = torch.device("cuda", torch.cuda.current_device())
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed)
    op = case["op"]
    if op == "batch":
        graphs = [_graph(s, gen) for s in _batch_shapes(case)]
        vtx = np.cumsum([0] + [n for n, _, _ in graphs]).astype(np.int64)
        nnz = np.cumsum([0] + [ci.numel() for _, _, ci in graphs]).astype(np.int64)
        ws = torch.empty(rcm.batched_workspace_bytes(len(graphs), int(vtx[-1]), int(nnz[-1])),
                         dtype=torch.uint8, device=dev)
        return {"case": case, "vtx": vtx, "nnz": nnz, "workspace": ws,
                "rowptr": torch.cat([rp for _, rp, _ in graphs]),
                "colidx": torch.cat([ci for _, _, ci in graphs])}
    n, rowptr, colidx = _graph(case, gen, case.get("banded", False))
    state = {"case": case, "rowptr": rowptr, "colidx": colidx}
    if op == "order":
        state["options"] = {k: case[k] for k in ("label_mode", "pp_variant", "reverse_mode",
                                                 "check_full") if case.get(k)}
        if case.get("tuned"):
            state["options"]["tuning_file"] = MI355X_TABLE
        if case.get("workspace"):
            state["workspace"] = torch.empty(rcm.workspace_bytes(n, colidx.numel()),
                                             dtype=torch.uint8, device=dev)
        return state
    state["vals"] = _normal(colidx.numel(), gen) if case["values"] else None
    if op == "spmv":
        state["x"] = _normal(n, gen)
        return state
    state["perm"], state["iperm"], _ = rcm.order(rowptr, colidx, return_iperm=True)
    state["workspace"] = torch.empty(
        apply.permute_workspace_bytes(n, colidx.numel(), case["values"]), dtype=torch.uint8,
        device=dev)
    return state


def run(state):
    op = state["case"]["op"]
    if op == "order":
        perm, iperm, stats = rcm.order(state["rowptr"], state["colidx"], return_iperm=True,
                                       workspace=state.get("workspace"), **state["options"])
        return perm, iperm, [stats[k] for k in STATS]
    if op == "batch":
        perm, stats = rcm.order_batched(state["vtx"], state["nnz"], state["rowptr"],
                                        state["colidx"], workspace=state["workspace"])
        return perm, np.array([[s[k] for k in STATS] for s in stats], dtype=np.int64)
    if op == "permute":
        return apply.permute(state["rowptr"], state["colidx"], state["perm"], state["iperm"],
                             state["vals"], workspace=state["workspace"])
    return apply.spmv(state["rowptr"], state["colidx"], state["x"], state["vals"])


def _size(case):
    """Vertices and (for random structures, expected) stored entries."""
    a, b, c = case["a"], case["b"], case["c"]
    if case["kind"] == "rgg":
        return a, 13 * a
    n = a * b * c
    edges = (a - 1) * b * c + a * (b - 1) * c + a * b * (c - 1)
    return n, n + (2 * edges if case["kind"] != "strip" else int(1.98 * edges))


def work(case):
    if case["op"] == "batch":
        sizes = [_size(s) for s in _batch_shapes(case)]
        n, nnz = sum(s[0] for s in sizes), sum(s[1] for s in sizes)
        return {"bytes": 4 * n + 4 * nnz + 4 * n, "flops": 0}
    n, nnz = _size(case)
    if case["op"] == "order":  # rows and columns in; the order and its inverse out
        return {"bytes": 4 * n + 4 * nnz + 8 * n, "flops": 0}
    value = 8 if case["values"] else 0
    if case["op"] == "permute":  # the matrix, the order and its inverse in; the matrix out
        return {"bytes": 2 * (4 * n + (4 + value) * nnz) + 8 * n, "flops": 0}
    return {"bytes": 4 * n + (4 + value) * nnz + 16 * n, "flops": 2 * nnz}


def exact(case, seed):
    """Orders and permuted matrices are whole numbers and copies; the product
    is summed here by plain torch in float64."""
    if case["op"] != "spmv":
        return None
    s = prepare(case, seed)
    rows = torch.repeat_interleave(torch.arange(s["x"].numel(), device=s["x"].device),
                                   (s["rowptr"][1:] - s["rowptr"][:-1]).long())
    terms = s["x"][s["colidx"].long()]
    if s["vals"] is not None:
        terms = terms * s["vals"]
    return torch.zeros_like(s["x"]).index_add_(0, rows, terms)
