"""Performance cases: graph generation as a program that uses this package
asks for it, through the public calls of `paper_1710_07565_amd`.

A case is a dict of plain values.  `kind` names the call (gnm, gnp, view,
skip, batch, rgg2d, rgg3d); `sized` says that the program lets the call
allocate its output and workspace, as a script does; otherwise it keeps the
output buffer and the workspace from call to call, as a generation loop or a
server does (where the edge total is random, with room for ten standard
deviations above its mean).  Only the seed of the graph differs between two
states of a case.

Every output is whole: edge lists as pairs of 32-bit words, totals, instance
offsets, and the points of the geometric graphs.
"""
import math

import torch

import paper_1710_07565_amd as kg
from paper_1710_07565_amd import workloads

DEVICE = "cuda"


def listed():
    return [
        # The smallest use: a test-sized graph in a script that lets the call
        # allocate (4,096 vertices; the size the package's own smoke run has).
        # Launch latency and host work are what it waits for.
        {"name": "gnm_directed_n12", "kind": "gnm", "n": 2**12, "m": 2**16, "directed": True, "chunks": 8, "sized": True},
        # A small job of a generation loop with kept buffers: the benchmark's
        # 2^16-vertex directed workload (8 MiB of edges).
        {"name": "gnm_directed_n16", "kind": "gnm", "n": 2**16, "m": 2**20, "directed": True, "chunks": 64, "sized": False},
        # An ordinary graph of odd size: sections that are no power of two and
        # tiles of every chunk ragged, so each edge's decode divides.
        {"name": "gnm_undirected_odd", "kind": "gnm", "n": 3000017, "m": 48000271, "directed": False, "chunks": 37, "sized": False},
        # The headline workload of the benchmark and the largest case.
        {"name": "gnm_undirected_n26", "kind": "gnm", "n": 2**26, "m": 2**31, "directed": False, "chunks": 256, "sized": False},
        # The benchmark's two G(n,p) workloads: many row chunks with a binomial
        # count each, and the undirected one with the heavier degree.
        {"name": "gnp_directed_n25", "kind": "gnp", "n": 2**25, "degree": 16.0, "directed": True, "chunks": 2**16},
        {"name": "gnp_undirected_n25", "kind": "gnp", "n": 2**25, "degree": 64.0, "directed": False, "chunks": 256},
        # One processing element's part of the headline graph: the edges
        # incident to one of its 256 sections.
        {"name": "view_undirected_n26", "kind": "view", "n": 2**26, "m": 2**31, "directed": False, "chunks": 256, "rank": 77},
        # A batch of uneven instances in one call, the mix that the batched
        # workload and the server draw.
        {"name": "batch_64", "kind": "batch", "count": 64, "log2n_lo": 10, "log2n_hi": 22, "mix": 20240101},
        # The geometric-skip sampler on the benchmark's parameters.
        {"name": "skip_directed_n25", "kind": "skip", "n": 2**25, "degree": 16.0, "directed": True, "chunks": 2**16},
        # Random geometric graphs: the benchmark's two-dimensional graph, an
        # ordinary one of odd size, and the benchmark's three-dimensional graph.
        {"name": "rgg2d_n26", "kind": "rgg2d", "n": 2**26, "factor": 0.55},
        {"name": "rgg2d_odd", "kind": "rgg2d", "n": 1000003, "factor": 0.55},
        {"name": "rgg3d_n26", "kind": "rgg3d", "n": 2**26, "factor": 0.55},
    ]


def _odd(rng, lo, hi):
    """An integer spread over [2^lo, 2^hi] by its logarithm, rarely a power of two."""
    return int(2.0 ** rng.uniform(lo, hi)) | (rng.random() < 0.5)


def _chunks(rng, n, edges, directed):
    """The paper's P: chunks of at least 4,096 expected edges, up to the
    benchmark's 2^16 row chunks or 256 sections."""
    most = max(1.0, edges / 4096.0)
    top = min(most, 2**16) if directed else min(math.sqrt(2.0 * most), 256)
    return max(1, min(int(2.0 ** rng.uniform(0.0, math.log2(max(top, 1.0)) + 1e-9)), n))


def draw(rng):
    kind = rng.choice(["gnm", "gnm", "gnp", "gnp", "view", "skip", "batch", "rgg2d", "rgg3d"])
    directed = rng.random() < 0.5
    if kind == "gnm":
        sized = rng.random() < 0.25
        n = _odd(rng, 12, 25.9)
        m = int(n * rng.uniform(2.0, 32.0))
        return {"kind": kind, "n": n, "m": m, "directed": directed, "chunks": _chunks(rng, n, m, directed), "sized": sized}
    if kind == "gnp":
        n = _odd(rng, 12, 25)
        d = rng.uniform(2.0, 32.0) if directed else rng.uniform(4.0, 64.0)
        e = n * d * (1.0 if directed else 0.5)
        return {"kind": kind, "n": n, "degree": d, "directed": directed, "chunks": _chunks(rng, n, e, directed)}
    if kind == "view":
        n = _odd(rng, 20, 25.9)
        m = int(n * rng.uniform(4.0, 32.0))
        P = max(2, _chunks(rng, n, m, False))
        return {"kind": kind, "n": n, "m": m, "directed": directed, "chunks": P, "rank": rng.randrange(P)}
    if kind == "skip":
        n = _odd(rng, 14, 25)
        d = rng.uniform(2.0, 16.0)
        e = n * d * (1.0 if directed else 0.5)
        return {"kind": kind, "n": n, "degree": d, "directed": directed, "chunks": _chunks(rng, n, e, directed)}
    if kind == "batch":
        return {"kind": kind, "count": int(2.0 ** rng.uniform(3, 7)), "log2n_lo": rng.randint(10, 12),
                "log2n_hi": rng.randint(20, 22), "mix": rng.randrange(1 << 30)}
    return {"kind": kind, "n": _odd(rng, 14, 25), "factor": rng.uniform(0.4, 0.65)}


def _slots(case):
    return case["n"] * (case["n"] - 1) // (1 if case["directed"] else 2)


def _p(case):
    """Edge probability of a mean out-degree (directed) or mean degree (undirected)."""
    return min(1.0, case["degree"] / (case["n"] - 1))


def _radius(case):
    """The radius recipe of the geometric experiments, 0.55 (ln n / n)^(1/d) at factor 0.55."""
    n, d = case["n"], 2 if case["kind"] == "rgg2d" else 3
    return case["factor"] * (math.log(n) / n) ** (1.0 / d)


def _view_mean(case):
    """Mean edge count of the case's view: its share of the slots times m."""
    n, P, r = case["n"], case["chunks"], case["rank"]
    h = (r + 1) * n // P - r * n // P
    incident = h * (n - 1) if case["directed"] else h * (n - h) + h * (h - 1) // 2
    return case["m"] * incident / _slots(case)


def _mean_edges(case):
    kind = case["kind"]
    if kind == "gnm":
        return float(case["m"])
    if kind in ("gnp", "skip"):
        return _p(case) * _slots(case)
    if kind == "view":
        return _view_mean(case)
    if kind == "batch":
        return float(sum(s.expected_edges() for s in _specs(case, 0)))
    f = kg.rgg2d_expected_edges if kind == "rgg2d" else kg.rgg3d_expected_edges
    return f(case["n"], _radius(case))


def _specs(case, seed):
    """The batch's instances: sizes, degrees, models and directions from the
    case, the instance seeds from the state's seed."""
    return workloads.batch_instances(case["count"], base_seed=seed, seed_fn=kg.instance_seed,
                                     log2n=(case["log2n_lo"], case["log2n_hi"]), rng_seed=case["mix"])


def _room(mean):
    """Edges a program reserves for a random total: ten standard deviations above the mean."""
    return int(mean + 10.0 * math.sqrt(mean) + 64)


def _edge_buffer(edges):
    # zeroed: what lies past the total stays as it was
    return torch.zeros((edges, 2), dtype=torch.int32, device=DEVICE).view(torch.uint32)


def _total():
    return torch.zeros(1, dtype=torch.int64, device=DEVICE).view(torch.uint64)


def _bytes(n):
    return torch.empty(max(int(n), 1), dtype=torch.uint8, device=DEVICE)


def prepare(case, seed):
    kind = case["kind"]
    seed = int(seed)
    state = {"case": case, "seed": seed}
    if kind == "batch":
        state["instances"] = [kg.Instance(s.n, s.model, s.directed, s.m, s.p, s.seed, s.chunks)
                              for s in _specs(case, seed)]
        mean = sum(_room(s.expected_edges()) for s in _specs(case, seed))
        state["arena"] = _edge_buffer(mean)
        state["offsets"] = torch.zeros(len(state["instances"]) + 1, dtype=torch.int64, device=DEVICE).view(torch.uint64)
        state["ws"] = _bytes(kg.workspace_bytes(state["instances"]))
        return state
    if kind in ("rgg2d", "rgg3d"):
        state["r"] = r = _radius(case)
        need = kg.rgg2d_workspace_bytes if kind == "rgg2d" else kg.rgg3d_workspace_bytes
        state["points"] = torch.zeros((case["n"], 2 if kind == "rgg2d" else 3), dtype=torch.float64, device=DEVICE)
        state["out"] = _edge_buffer(int(_mean_edges(case) * 1.02) + 65536)
        state["total"] = _total()
        state["ws"] = _bytes(need(case["n"], r))
        return state
    if not case.get("sized", False):
        P, directed = case["chunks"], case["directed"]
        if kind == "skip":
            need = kg.gnp_skip_workspace_bytes(case["n"], _p(case), directed, P)
        else:
            gnp = kind == "gnp"
            need = kg.workspace_bytes([kg.Instance(case["n"], kg.GNP if gnp else kg.GNM, directed, 0 if gnp else case["m"],
                                                   _p(case) if gnp else 0.0, seed, P, case.get("rank", -1) + 1)])
        state["ws"] = _bytes(need)
        state["out"] = _edge_buffer(case["m"] if kind == "gnm" else _room(_mean_edges(case)))
        state["total"] = _total()
    return state


def _plain(*tensors):
    """The outputs as signed words of the same width (the same bits)."""
    signed = {torch.uint32: torch.int32, torch.uint64: torch.int64}
    return [t.view(signed[t.dtype]) if t.dtype in signed else t for t in tensors]


def run(state):
    case, seed = state["case"], state["seed"]
    kind = case["kind"]
    if kind == "batch":
        arena, offsets = kg.batch(state["instances"], arena=state["arena"], offsets=state["offsets"], workspace=state["ws"])
        return _plain(arena, offsets)
    if kind in ("rgg2d", "rgg3d"):
        call = kg.rgg2d if kind == "rgg2d" else kg.rgg3d
        return _plain(*call(case["n"], state["r"], seed=seed, points=state["points"], out=state["out"],
                            total=state["total"], workspace=state["ws"]))
    directed, P = case["directed"], case["chunks"]
    if kind == "gnm":
        if case["sized"]:
            return _plain(kg.gnm(case["n"], case["m"], directed=directed, seed=seed, chunks=P))
        return _plain(kg.gnm(case["n"], case["m"], directed=directed, seed=seed, chunks=P, out=state["out"],
                             workspace=state["ws"]))
    kept = {"out": state["out"], "total": state["total"], "workspace": state["ws"]}
    if kind == "view":
        got = kg.pe_view(case["n"], case["rank"], P, directed=directed, m=case["m"], seed=seed, **kept)
    elif kind == "gnp":
        got = kg.gnp(case["n"], _p(case), directed=directed, seed=seed, chunks=P, **kept)
    else:
        got = kg.gnp_skip(case["n"], _p(case), directed=directed, seed=seed, chunks=P, **kept)
    return _plain(*got)


def work(case):
    """Bytes: every edge (two 32-bit ids) and point written once; the inputs
    are a few numbers.  Operations: a geometric edge's own distance test (5
    in two dimensions, 8 in three); the random graphs need no arithmetic that
    their definition counts."""
    edges = _mean_edges(case)
    if case["kind"] in ("rgg2d", "rgg3d"):
        d = 2 if case["kind"] == "rgg2d" else 3
        return {"bytes": 8.0 * edges + 8.0 * d * case["n"], "flops": (3 * d - 1) * edges}
    return {"bytes": 8.0 * edges, "flops": 0.0}


def exact(case, seed):
    """None: edges, totals and offsets are whole numbers, and the points are
    random draws whose bits the generator's streams define; none of them
    approximates a value of real arithmetic."""
    return None
