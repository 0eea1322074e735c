"""The work a program gives this library, as cases that can be timed.

A case names an input (its generator and sizes) and how it is coloured:

``once``    a graph seen for the first time goes through ``gc.color``: bound, checked, coloured, released.
``color``   a graph bound once (``gc.Graph``) is coloured, and its rounds and colours are read.
``batch``   a packed batch of graphs in one launch (``gc.color_batch``).
``steps``   the same batch advanced eight rounds at a time (``gc.batch_step``), as a server does.

Inputs are drawn on the GPU from the seed: Erdos-Renyi (``er``), R-MAT with (.57, .19, .19, .05) (``rmat``), a
27-point stencil under a random numbering (``stencil``), and batches of Erdos-Renyi graphs of mixed sizes.
"""
import math

import numpy as np
import torch

from paper_1509_08267_amd import gc

DEVICE = "cuda:0"


def _color(gen, algorithm="push", rows_sorted=True, i64=False, partitions=0, **sizes):
    return {"kind": "color", "gen": gen, "algorithm": algorithm, "rows_sorted": rows_sorted, "i64": i64,
            "partitions": partitions, **sizes}


def _batch(kind, graphs, nmin=100, nmax=50_000, dmin=4.0, dmax=64.0):
    return {"kind": kind, "gen": "batch", "graphs": graphs, "nmin": nmin, "nmax": nmax, "dmin": dmin, "dmax": dmax}


def listed():
    return [
        # one small graph from a caller that sees it once (a register-allocation or timetabling size): set-up counts
        {"name": "once_er_2k", "kind": "once", "gen": "er", "n": 2_000, "m": 20_000, "rows_sorted": True, "i64": False},
        # the smallest bound graph of the benchmark: a dozen rounds of little work each
        {"name": "er_10k", **_color("er", n=10_000, m=100_000)},
        # the benchmark's default workload
        {"name": "er_1m", **_color("er", n=1 << 20, m=1 << 24)},
        # an odd size from an edge list that nobody sorted
        {"name": "er_300k_unsorted", **_color("er", rows_sorted=False, n=300_007, m=2_700_011)},
        # a regular mesh, nothing but short rows (finite-element assembly, smoothers)
        {"name": "stencil_160", **_color("stencil", side=160)},
        # the stand-in for the social networks of the paper's experiments: hubs, hundreds of rounds, 64-bit offsets
        {"name": "rmat_22", **_color("rmat", scale=22, edge_factor=16, i64=True)},
        # a dense interference graph: hundreds of colours, every row a wavefront's work
        {"name": "dense_8k", **_color("er", n=8_000, m=4_000_000)},
        # the paper's sequential baseline, computed in parallel, on the uniform and on the skewed input
        {"name": "seq_er_1m", **_color("er", algorithm="seq", n=1 << 20, m=1 << 24)},
        {"name": "seq_rmat_20", **_color("rmat", algorithm="seq", scale=20, edge_factor=16)},
        # the paper's own algorithm, read literally, with p blocks
        {"name": "blocks_er_1m", **_color("er", algorithm="blocks", partitions=16_384, n=1 << 20, m=1 << 24)},
        # a server's resident set, advanced in steps
        {"name": "steps_512", **_batch("steps", 512)},
        # the benchmark's batch
        {"name": "batch_4096", **_batch("batch", 4_096)},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["once", "er", "er", "er", "rmat", "rmat", "stencil", "dense", "seq", "blocks", "steps", "batch", "batch"])
    i64 = rng.random() < 0.3
    rows_sorted = rng.random() < 0.75
    algorithm = "pull" if rng.random() < 0.15 else "push"
    if kind == "once":
        n = _log(rng, 500, 200_000)
        return {"kind": "once", "gen": "er", "n": n, "m": int(n * rng.uniform(2.0, 16.0)), "rows_sorted": rows_sorted, "i64": i64}
    if kind in ("er", "seq", "blocks"):
        if kind == "seq" and rng.random() < 0.4:
            return _color("rmat", algorithm="seq", i64=i64, scale=rng.randint(12, 19), edge_factor=rng.randint(8, 16))
        n = _log(rng, 1_000, 1 << 20) | 1
        m = int(n * rng.uniform(2.0, 16.0))
        if kind == "blocks":
            return _color("er", algorithm="blocks", i64=i64, partitions=_log(rng, max(64, n // 128), max(65, n // 16)), n=n, m=m)
        return _color("er", algorithm="seq" if kind == "seq" else algorithm, rows_sorted=rows_sorted, i64=i64, n=n, m=m)
    if kind == "rmat":
        return _color("rmat", algorithm=algorithm, rows_sorted=rows_sorted, i64=i64, scale=rng.randint(12, 21), edge_factor=rng.randint(8, 16))
    if kind == "stencil":
        return _color("stencil", algorithm=algorithm, rows_sorted=rows_sorted, i64=i64, side=_log(rng, 12, 150))
    if kind == "dense":
        n = _log(rng, 1_000, 8_000) | 1
        return _color("er", algorithm=algorithm, i64=i64, n=n, m=int(n * n * rng.uniform(0.02, 0.06)))
    nmax = _log(rng, 2_000, 50_000)
    return _batch(kind, _log(rng, 1, 2_048), nmax=nmax, dmin=4.0, dmax=round(rng.uniform(8.0, 64.0), 1))


# ------------------------------------------------------------------ inputs --

def _generator(seed):
    g = torch.Generator(device=DEVICE)
    g.manual_seed(seed)
    return g


def _edges_er(case, gen):
    n = case["n"]
    return n, torch.randint(n, (2, case["m"]), generator=gen, device=DEVICE)


def _edges_rmat(case, gen):
    scale, count = case["scale"], case["edge_factor"] << case["scale"]
    uv = torch.zeros((2, count), dtype=torch.int64, device=DEVICE)
    for _ in range(scale):
        x = torch.rand(count, generator=gen, device=DEVICE)
        u = x >= 0.76                       # a + b
        v = ((x >= 0.57) & ~u) | (x >= 0.95)  # b, or d
        uv[0].mul_(2).add_(u)
        uv[1].mul_(2).add_(v)
    return 1 << scale, uv


def _edges_stencil(case, gen):
    side = case["side"]
    n = side ** 3
    name = torch.randperm(n, generator=gen, device=DEVICE)
    cell = torch.arange(n, device=DEVICE).view(side, side, side)
    pairs = []
    for d in range(14, 27):  # one of each two opposite directions
        dx, dy, dz = d // 9 - 1, d // 3 % 3 - 1, d % 3 - 1
        at = tuple(slice(max(0, -s), side - max(0, s)) for s in (dx, dy, dz))
        to = tuple(slice(max(0, s), side - max(0, -s)) for s in (dx, dy, dz))
        pairs.append(torch.stack([name[cell[at].reshape(-1)], name[cell[to].reshape(-1)]]))
    return n, torch.cat(pairs, 1)


def _rows(n, uv):
    """Ascending CSR (counts, columns) of the simple undirected graph on these pairs."""
    uv = uv[:, uv[0] != uv[1]]
    key = torch.unique(torch.minimum(uv[0], uv[1]) * n + torch.maximum(uv[0], uv[1]))
    a, b = key // n, key % n
    del uv, key
    key = torch.sort(torch.cat([a * n + b, b * n + a]))[0]
    del a, b
    row = key // n
    col = (key - row * n).to(torch.int32)
    return torch.bincount(row, minlength=n), col


def _graph(case, seed):
    gen = _generator(seed)
    n, uv = {"er": _edges_er, "rmat": _edges_rmat, "stencil": _edges_stencil}[case["gen"]](case, gen)
    deg, col = _rows(n, uv)
    if not case["rows_sorted"]:
        row = torch.repeat_interleave(torch.arange(n, device=DEVICE), deg)
        key = (row << 31) | torch.randint(1 << 31, (col.numel(),), generator=gen, device=DEVICE)
        col = col[torch.sort(key)[1]]
    rp = torch.zeros(n + 1, dtype=torch.int64, device=DEVICE)
    torch.cumsum(deg, 0, out=rp[1:])
    return rp if case["i64"] else rp.to(torch.int32), col.contiguous()


def _graphs(case, seed):
    """A packed batch: offsets (device and host), local row pointers, local columns.  The sizes are the case's own;
    the seed draws the edges."""
    G = case["graphs"]
    rs = np.random.RandomState(G + case["nmax"])
    ns = np.exp(rs.uniform(math.log(case["nmin"]), math.log(case["nmax"]), G)).astype(np.int64)
    ms = (ns * rs.uniform(case["dmin"], case["dmax"], G) / 2).astype(np.int64)
    gen = _generator(seed)
    degs, cols = [], []
    voff = np.concatenate([[0], np.cumsum(ns)])
    g0 = 0
    while g0 < G:  # a group of graphs of about 2^25 pairs at a time
        g1 = g0 + 1
        while g1 < G and ms[g0:g1 + 1].sum() <= 1 << 25:
            g1 += 1
        n_d = torch.from_numpy(ns[g0:g1]).to(DEVICE)
        base = torch.from_numpy(voff[g0:g1] - voff[g0]).to(DEVICE)
        of = torch.repeat_interleave(torch.arange(g1 - g0, device=DEVICE), torch.from_numpy(ms[g0:g1]).to(DEVICE))
        uv = (torch.rand((2, of.numel()), generator=gen, device=DEVICE, dtype=torch.float64) * n_d[of]).to(torch.int64) + base[of]
        n = int(voff[g1] - voff[g0])
        deg, col = _rows(n, uv)
        first = torch.repeat_interleave(base, n_d)  # of each vertex, then of each entry
        cols.append(col - torch.repeat_interleave(first, deg).to(torch.int32))
        degs.append(deg)
        g0 = g1
    deg, col = torch.cat(degs), torch.cat(cols)
    rp = torch.zeros(deg.numel() + 1, dtype=torch.int64, device=DEVICE)
    torch.cumsum(deg, 0, out=rp[1:])
    v_d = torch.from_numpy(voff).to(DEVICE)
    eoff = rp[v_d]
    idx = torch.arange(G, device=DEVICE)
    of = torch.repeat_interleave(idx, torch.from_numpy(ns).to(DEVICE))
    local = torch.empty(deg.numel() + G, dtype=torch.int32, device=DEVICE)
    local[torch.arange(deg.numel(), device=DEVICE) + of] = (rp[:-1] - eoff[of]).to(torch.int32)
    local[v_d[1:] + idx] = (eoff[1:] - eoff[:-1]).to(torch.int32)
    return {"voff": v_d, "eoff": eoff, "rp": local, "ci": col, "voff_host": voff, "eoff_host": eoff.cpu().numpy()}


# -------------------------------------------------------------- the passes --

def prepare(case, seed):
    if case["gen"] == "batch":
        s = {"kind": case["kind"], **_graphs(case, seed)}
        if case["kind"] == "steps":
            rows = [(int(v + g), int(e), int(v), int(s["voff_host"][g + 1] - v))
                    for g, (v, e) in enumerate(zip(s["voff_host"][:-1], s["eoff_host"][:-1]))]
            s["fresh"] = torch.from_numpy(gc.desc_array(rows).view(np.uint8)).to(DEVICE)
            s["colors"] = torch.empty(int(s["voff_host"][-1]), dtype=torch.int32, device=DEVICE)
            s["workspace"] = torch.empty(gc.gc_batch_step_workspace_bytes(case["graphs"], 0), dtype=torch.uint8, device=DEVICE)
        return s
    rp, ci = _graph(case, seed)
    if case["kind"] == "once":
        return {"kind": "once", "rp": rp, "ci": ci, "rows_sorted": case["rows_sorted"]}
    options = {"algorithm": case["algorithm"]}
    if case["partitions"]:
        options["partitions"] = case["partitions"]
    return {"kind": "color", "graph": gc.Graph(rp, ci, rows_sorted=case["rows_sorted"], **options)}


def run(state):
    if state["kind"] == "once":
        return {"colors": gc.color(state["rp"], state["ci"], validate=True, rows_sorted=state["rows_sorted"])}
    if state["kind"] == "color":
        colors = state["graph"].color()
        rounds, num_colors = state["graph"].stats()
        return {"colors": colors, "rounds": rounds, "num_colors": num_colors}
    if state["kind"] == "batch":
        colors, rounds = gc.color_batch(state["voff"], state["eoff"], state["rp"], state["ci"],
                                        voff_host=state["voff_host"], eoff_host=state["eoff_host"])
        return {"colors": colors, "rounds": rounds}
    descs = state["fresh"].clone()
    for rounds in (8, 8, 8, 0):  # three steps, then whatever is left
        gc.batch_step(descs, state["rp"], state["ci"], state["colors"], rounds, workspace=state["workspace"])
    table = descs.view(torch.int32).view(-1, 10)  # gc_graph_desc: rounds and active are its words 7 and 8
    return {"colors": state["colors"], "rounds": table[:, 7], "active": table[:, 8]}


def _sizes(case):
    """(graphs, vertices, CSR entries) a case has on average."""
    if case["gen"] == "batch":
        span = math.log(case["nmax"] / case["nmin"])
        n = case["graphs"] * (case["nmax"] - case["nmin"]) / span
        return case["graphs"], n, n * (case["dmin"] + case["dmax"]) / 2
    if case["gen"] == "er":
        pairs = case["n"] * (case["n"] - 1) / 2
        return 1, case["n"], 2 * pairs * -math.expm1(-case["m"] / pairs)
    if case["gen"] == "rmat":  # about 4% of the samples are loops or repeats at scale 22, more at smaller ones
        return 1, 1 << case["scale"], 2 * 0.9 * (case["edge_factor"] << case["scale"])
    return 1, case["side"] ** 3, (3 * case["side"] - 2) ** 3 - case["side"] ** 3


def work(case):
    """Row pointers and columns read once, colours written once; there is no floating-point work."""
    graphs, n, entries = _sizes(case)
    return {"bytes": (n + graphs) * (8 if case.get("i64") else 4) + 4 * entries + 4 * n, "flops": 0}


# ---------------------------------------------------------- the definition --

def _define(n, row, col, sequential, most=1024):
    """(colour, round) of every vertex by the definition: rounds of First Fit over the final neighbours, where the
    lower id of a conflicting pair keeps its colour, or (sequential) a vertex waits for all its lower neighbours."""
    color = torch.full((n,), -1, dtype=torch.int64, device=DEVICE)
    when = torch.zeros(n, dtype=torch.int64, device=DEVICE)
    k = min(most, int(torch.bincount(row, minlength=n).max()) + 1 if row.numel() else 1)
    taken = torch.zeros((n, k), dtype=torch.bool, device=DEVICE)
    number = torch.arange(k, device=DEVICE)
    left, r = torch.arange(n, device=DEVICE), 0
    tent = torch.zeros(n, dtype=torch.int64, device=DEVICE)
    while left.numel():
        r += 1
        tent[left] = torch.where(taken[left], k, number).amin(1)
        lose = torch.zeros(n, dtype=torch.bool, device=DEVICE)
        lower = col < row
        lose[row[lower if sequential else lower & (tent[row] == tent[col])]] = True
        won = left[~lose[left]]
        if int(tent[won].max()) >= k:
            return None, None
        color[won], when[won] = tent[won], r
        told = (color[row] >= 0) & (color[col] < 0)
        taken[col[told], color[row[told]]] = True
        both = (color[row] < 0) & (color[col] < 0)
        row, col, left = row[both], col[both], left[lose[left]]
    return color, when


def exact(case, seed):
    _, n, entries = _sizes(case)
    if entries > 4e7 or case.get("algorithm") == "blocks":
        return None
    if case["gen"] == "batch":
        s = _graphs(case, seed)
        G, n = case["graphs"], int(s["voff_host"][-1])
        of = torch.repeat_interleave(torch.arange(G, device=DEVICE), s["voff"].diff())
        v = torch.arange(n, device=DEVICE)
        deg = (s["rp"][v + of + 1] - s["rp"][v + of]).long()
        row = torch.repeat_interleave(v, deg)
        color, when = _define(n, row, s["ci"].long() + s["voff"][of[row]], False)
        if color is None:
            return None
        rounds = torch.zeros(G, dtype=torch.int64, device=DEVICE).scatter_reduce(0, of, when, "amax")
        out = {"colors": color, "rounds": rounds}
        return {**out, "active": torch.zeros_like(rounds)} if case["kind"] == "steps" else out
    rp, ci = _graph(case, seed)
    n = rp.numel() - 1
    row = torch.repeat_interleave(torch.arange(n, device=DEVICE), rp.long().diff())
    if case["gen"] == "rmat" and n > 1 << 17:  # hundreds of colours: the table of taken ones gets too large
        return None
    color, when = _define(n, row, ci.long(), case.get("algorithm") == "seq")
    if color is None:
        return None
    if case["kind"] == "once":
        return {"colors": color}
    return {"colors": color, "rounds": int(when.max()), "num_colors": int(color.max()) + 1}
