"""What a user of the placement library has it do, as measurable cases.

A case is one pass of the library's public entry points over a synthetic
operator graph (the generators of ``workloads``: layered random DAGs,
transformer training graphs at micro-op granularity, inception-like fork/join
modules), sizes between two thousand and a million nodes.  Five kinds of work:

- ``plan``: a placement from nothing: levels, b-level and priority order,
  clustering, Adjusting Placement, and the makespan of the result;
- ``score``: evaluate a placement in hand.  K = 1: b-level, t-level, critical
  path and the full schedule (start and finish times).  K > 1: the makespans
  of K candidate placements, a clustering with 5 % of its clusters moved;
- ``models``: the makespan of K placements under a device model (first-fit
  insertion, transfers as tasks or as blocking operations), on identical or
  heterogeneous devices;
- ``extend``: Adjusting Placement on heterogeneous devices and links with
  co-location groups inside the algorithm;
- ``baseline``: the comparison a placement is judged by: the depth-first
  orders, greedy clustering, Order-Place and the communication ratio's sums.

Every output is a whole number or a byte (times are int64 nanoseconds), so
nothing is rounded and outputs are compared exactly.
"""
from __future__ import annotations

import copy
import functools
import math

import numpy as np
import torch

import paper_2208_00184_amd as cel
from workloads import graphs, perturb_placements

DEVICE = "cuda:0"

# device-model bits
FIFO, INSERT, TASKS, BLOCK = 0, cel.MODEL_INSERT, cel.MODEL_COMM_TASKS, cel.MODEL_COMM_BLOCK


def _layered(layers, width, back, D):
    return dict(graph="layered", layers=layers, width=width, back=back, D=D)


def _transformer(blocks, hidden, heads, tiles, D):
    return dict(graph="transformer", blocks=blocks, hidden=hidden, heads=heads, tiles=tiles, D=D)


def _inception(modules, D):
    return dict(graph="inception", modules=modules, D=D)


def listed():
    # The sizes are the repository's own configurations: layered-2k,
    # transformer-24 (20k nodes), inception-600 (54k), layered-200k and
    # transformer-96 (1.07M nodes, 10,565 levels).
    tf96 = _transformer(96, 8192, 64, 32, 16)
    inc600 = _inception(600, 8)
    return [
        # the smallest graph a user plans: launches, round trips and latency
        dict(name="plan-layered-2k", work="plan", R=200, **_layered(64, 32, 4, 4)),
        # ordinary model graphs: deep and narrow; many joins
        dict(name="plan-transformer-24", work="plan", R=200, **_transformer(24, 1024, 16, 1, 4)),
        dict(name="plan-inception-600", work="plan", R=200, **inc600),
        # a shallow random graph of wide levels
        dict(name="plan-layered-200k", work="plan", R=200, **_layered(400, 500, 8, 8)),
        # the largest graph
        dict(name="plan-transformer-96", work="plan", R=200, **tf96),
        # one placement evaluated in full: the inner step of a search
        dict(name="score-transformer-96", work="score", K=1, R=200, **tf96),
        # a population of candidates scored in one call: deep graph, few; wide graph, many
        dict(name="score64-transformer-96", work="score", K=64, R=200, **tf96),
        dict(name="score1024-layered-200k", work="score", K=1024, R=200, **_layered(400, 500, 8, 8)),
        # the chosen placement checked against contended links
        dict(name="tasks-transformer-96", work="models", model=TASKS, hetero=False, K=1, R=200, **tf96),
        # a few placements of a mixed machine under the insertion schedule
        dict(name="insert16-inception-600", work="models", model=INSERT, hetero=True, K=16, R=200, **inc600),
        # a mixed machine planned with co-location groups
        dict(name="extend-transformer-96", work="extend", R=200, **tf96),
        # the baselines of a comparison
        dict(name="baseline-inception-600", work="baseline", R=200, **inc600),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_graph(rng, most):
    """A graph of up to about `most` nodes, sizes spread over their logarithm."""
    n = _log(rng, 1000, most)
    D = rng.choice([2, 3, 4, 6, 8, 12, 16, 24, 32, 64])
    kind = rng.choice(["layered", "narrow", "tiled", "inception"])
    if kind == "tiled" and n >= 2 * 11150:  # 11,150 nodes a block
        return _transformer(n // 11150, 8192, 64, 32, D)
    if kind == "narrow" or kind == "tiled":  # 830 nodes a block; deep
        return _transformer(max(1, min(n // 830, 120)), 1024, 16, 1, D)
    if kind == "inception":  # 90 nodes a module
        return _inception(max(8, min(n // 90, 1200)), D)
    width = max(_log(rng, 8, max(9, min(700, n // 20))), n // 4000)  # at most about 4,000 layers
    return _layered(max(5, n // width), width, rng.randint(2, 12), D)


def draw(rng):
    work = rng.choice(["plan", "plan", "plan", "score", "batch", "batch", "models", "extend", "baseline"])
    R = rng.choice([64, 100, 150, 200, 200, 200, 257, 400])
    if work == "plan":
        return dict(work="plan", R=R, **_draw_graph(rng, 1000000))
    if work == "score":
        return dict(work="score", K=1, R=R, **_draw_graph(rng, 1000000))
    if work == "batch":
        g = _draw_graph(rng, 300000)
        return dict(work="score", K=_log(rng, 2, 400), R=R, **g)
    if work == "models":
        g = _draw_graph(rng, 150000)
        return dict(work="models", model=rng.choice([FIFO, INSERT, TASKS, TASKS, INSERT | TASKS, BLOCK]),
                    hetero=rng.random() < 0.4, K=rng.choice([1, 1, 1, 2, 4, 16, 33]), R=R, **g)
    if work == "extend":
        return dict(work="extend", R=R, **_draw_graph(rng, 500000))
    return dict(work="baseline", R=R, **_draw_graph(rng, 300000))


@functools.lru_cache(maxsize=3)
def _structure(key):
    """The graph of a case with the costs of its first profile."""
    case = dict(key)
    D = case["D"]
    if case["graph"] == "layered":
        return graphs._layered_config(5, 0, case["layers"], case["width"], case["back"], D)
    if case["graph"] == "transformer":
        wide = case["tiles"] > 1
        return graphs._transformer(4 if wide else 2, 0, case["hidden"], case["heads"], case["tiles"],
                                   case["blocks"], D, 16, 10 * D, 50 if wide else 25, 2000 if wide else 3000)
    return graphs._inception(3, 0, case["modules"])


def _graph_of(case):
    return _structure(tuple(sorted((k, v) for k, v in case.items()
                                   if k not in ("name", "work", "model", "hetero", "K", "R"))))


def _workload(case, seed):
    """The case's graph with the costs of another profile of the same program:
    every time and size off by its own factor."""
    base = _graph_of(case)
    rng = np.random.default_rng([case["D"], seed])
    wl = copy.copy(base)
    wl.w = np.maximum(1, np.rint(base.w * rng.lognormal(0.0, 0.4, base.n))).astype(np.int64)
    wl.ob = np.maximum(1, np.rint(base.ob * rng.lognormal(0.0, 0.4, base.n))).astype(np.int64)
    wl.mem = 2 * wl.ob
    return wl


def _devices(wl, D):
    """Memory caps are a share of 1.6 / D of the total each, as the
    configurations have it (0.35 of it for D = 4, 0.2 for 8, 0.1 for 16)."""
    return cel.Devices(D, np.full(D, int(wl.mem.sum()) * 16 // (10 * D), np.int64), wl.bw, wl.lat)


class _State:
    """A graph on the GPU, its devices, and what the program has computed of it before."""


def _plan(g, d, R):
    """The whole path, as a program that wants a placement calls it."""
    lev, oid, lp, L = cel.topo_levels(g)
    bl, _, prio, cp = cel.blevel(g, d, lev, lp, oid, L)
    cid, C, cut = cel.cluster(g, d, prio, R, -1)
    cdev, ndev, span, be = cel.place(g, d, cid, C)
    return dict(level=lev, order_id=oid, level_ptr=lp, L=L, blevel=bl, prio=prio, cp=cp, cluster_id=cid, C=C,
                cut=cut, cluster_dev=cdev, node_dev=ndev, coarse_makespan=span, best_effort=be)


def _hetero(d):
    """Half of the devices twice as slow; links inside a pair of devices twice as fast."""
    D = d.D
    return dict(tmul=[1024 if x < D // 2 else 2048 for x in range(D)],
                bw=[[2 * d.bw if x // 2 == y // 2 else d.bw for y in range(D)] for x in range(D)],
                lat=[[d.lat // 2 if x // 2 == y // 2 else d.lat for y in range(D)] for x in range(D)])


def prepare(case, seed):
    s = _State()
    wl = _workload(case, seed)
    s.case, s.g, s.d = case, cel.Graph.from_arrays(wl, DEVICE), _devices(wl, case["D"])
    if case["work"] == "plan":
        return s
    p = _plan(s.g, s.d, case["R"])
    if case["work"] == "extend":  # the clusters of the first profile, placed under the costs of this one
        base = _graph_of(case)
        p0 = _plan(cel.Graph.from_arrays(base, DEVICE), _devices(base, case["D"]), case["R"])
        p["cluster_id"], p["C"] = p0["cluster_id"], p0["C"]
    s.level, s.order_id, s.level_ptr, s.L, s.prio = (p[k] for k in ("level", "order_id", "level_ptr", "L", "prio"))
    s.cluster_id, s.C = p["cluster_id"], p["C"]
    if case["work"] == "baseline":
        _, s.tlevel, _, _ = cel.blevel(s.g, s.d, s.level, s.level_ptr, s.order_id, s.L, want_tlevel=True)
        s.blevel = p["blevel"]
    if case["work"] in ("score", "models"):
        s.node_dev = p["node_dev"]
        if case["K"] > 1:  # candidates: the placement with 5 % of its clusters moved
            maps = torch.from_numpy(perturb_placements(p["cluster_dev"].cpu().numpy(), s.d.D, case["K"], seed))
            s.node_dev = maps.to(DEVICE)[:, s.cluster_id.long()].contiguous()
    s.hetero = _hetero(s.d) if case["work"] == "extend" or case.get("hetero") else {}
    if case["work"] == "extend":  # groups of 4 over a tenth of the nodes
        s.G = wl.n // 40
        group = np.full(wl.n, -1, np.int32)
        pick = np.random.default_rng([seed, 17]).permutation(wl.n)[:4 * s.G]
        group[pick] = np.repeat(np.arange(s.G, dtype=np.int32), 4)
        s.group = torch.from_numpy(group).to(DEVICE)
    return s


def run(s):
    case, g, d = s.case, s.g, s.d
    if case["work"] == "plan":
        p = _plan(g, d, case["R"])
        ms, _, _ = cel.makespan(g, d, p["prio"], p["level"], p["level_ptr"], p["L"], p["node_dev"])
        p["makespan"] = ms
        del p["cluster_dev"]  # node_dev says it, node by node
        return p
    if case["work"] == "score" and case["K"] == 1:
        bl, tl, prio, cp = cel.blevel(g, d, s.level, s.level_ptr, s.order_id, s.L, want_tlevel=True)
        ms, start, finish = cel.makespan(g, d, prio, s.level, s.level_ptr, s.L, s.node_dev, want_times=True)
        return dict(blevel=bl, tlevel=tl, prio=prio, cp=cp, makespan=ms, start=start, finish=finish)
    if case["work"] == "score":
        return cel.makespan(g, d, s.prio, s.level, s.level_ptr, s.L, s.node_dev)[0]
    if case["work"] == "models":
        ms, start, finish = cel.makespan_model(g, d, s.prio, s.node_dev, case["model"], want_times=case["K"] == 1,
                                               **s.hetero)
        return dict(makespan=ms, start=start, finish=finish)
    if case["work"] == "extend":
        cdev, ndev, span, be, fin = cel.place_ext(g, d, s.cluster_id, s.C, group=s.group, n_groups=s.G, **s.hetero)
        return dict(cluster_dev=cdev, node_dev=ndev, coarse_makespan=span, best_effort=be, cluster_fin=fin)
    cpd = cel.cpd_order(g, s.blevel, s.tlevel)
    dfs = cel.dfs_order(g)
    cid, C, cut = cel.cluster(g, d, cpd, case["R"], -1, cel.CLUSTER_GREEDY)
    cdev, ndev, be = cel.order_place(g, d, cid, C)
    ms, _, _ = cel.makespan(g, d, s.prio, s.level, s.level_ptr, s.L, ndev)
    return dict(cpd=cpd, dfs=dfs, cluster_id=cid, C=C, cut=cut, node_dev=ndev, best_effort=be, ccr=cel.comm_sums(g, d),
                ccr_fused=cel.comm_sums(g, d, cid), makespan=ms)


def work(case):
    """Bytes of the inputs read once and the outputs written once; integer
    operations: an add and a maximum for each edge of each recurrence, and for
    the clustering three for each of R candidates of each node."""
    n, m = _graph_of(case).n, _graph_of(case).m
    K, R = case.get("K", 1), case["R"]
    graph = 8 * (n + 1) + 8 * m + 24 * n
    if case["work"] == "plan":  # level, order, b-level, priority order, cluster, device
        return dict(bytes=graph + 4 * n + 4 * n + 8 * n + 4 * n + 4 * n + n, flops=8 * m + 3 * n * R)
    if case["work"] == "score" and K == 1:
        return dict(bytes=graph + 9 * n + 8 * n + 8 * n + 4 * n + 16 * n, flops=6 * m)
    if case["work"] == "score":  # order, levels, K device maps
        return dict(bytes=graph + 8 * n + K * (n + 8), flops=2 * K * m)
    if case["work"] == "models":
        return dict(bytes=graph + 4 * n + K * (n + 8) + (16 * n if K == 1 else 0), flops=2 * K * m)
    if case["work"] == "extend":
        return dict(bytes=graph + 8 * n + n, flops=2 * m * case["D"])
    return dict(bytes=graph + 16 * n + 4 * n + 4 * n + 4 * n + n, flops=6 * m)


def tolerance(case):
    return "exact"  # whole numbers throughout


def exact(case, seed):
    return None  # whole numbers throughout: no output is an approximation of a real value
