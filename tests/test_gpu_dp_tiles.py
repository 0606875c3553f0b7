"""GPU parity of the clustering DP's tiled policy iteration against the CPU
oracle, tolerance 0: every split of the candidates over waves (16 ways on the
smallest graphs to one), three and five targets per lane, tiles and windows
that end inside a wave, windows of one to 4,096 positions, and memory caps
that cut them."""
from __future__ import annotations

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # collected on CPU, skipped there
    pytest.skip("needs a ROCm GPU", allow_module_level=True)

import paper_2208_00184_amd as cel  # noqa: E402
from oracle import oracle as O  # noqa: E402
from workloads import from_edges, graphs  # noqa: E402

DEV = "cuda:0"


def check(wl, order, R, M, policy=True):
    ref = O.cluster(wl, order, R, M)
    g, d = cel.Graph.from_arrays(wl, DEV), cel.Devices.from_arrays(wl)
    cid, C, cut = cel.cluster(g, d, torch.from_numpy(np.ascontiguousarray(order, np.int32)).to(DEV), R, M)
    info = cel.cluster_info()
    print(f"[dp] n={wl.n} R={R} M={M} {info}", flush=True)
    assert (C, cut) == (ref[1], ref[2])
    assert np.array_equal(cid.cpu().numpy(), ref[0])
    if policy:
        assert info[0] == 0  # by policy iteration


def near_dag(n, seed, reach, fan):
    """Edges to targets up to `reach` positions ahead (duplicates kept), ids in order."""
    rng = np.random.default_rng([seed, n])
    src = np.repeat(np.arange(n - 1), rng.integers(0, fan + 1, n - 1))
    dst = np.minimum(n - 1, src + rng.integers(1, reach + 1, src.size))
    ob = rng.integers(0, 3000, n) * (rng.random(n) < 0.9)
    return from_edges(n, np.stack([src, dst], 1), rng.integers(0, 50, n), ob, 2,
                      [int(2 * ob.sum()) + 1] * 2, 7, 3)


# targets per lane and waves per target follow from n at 256 workgroups:
# up to 16,384 -> 16 waves, 32,768 -> 8, 65,536 -> 4, 131,072 -> 2, 262,144 -> 1,
# above three targets per lane (five above 786,432: the transformer tests)
@pytest.mark.parametrize("n", [3072, 3073, 6001, 16384, 16385, 20011, 32769, 65537, 131073, 262145, 270001])
def test_sizes(n):
    wl = near_dag(n, 1, 90, 3)
    check(wl, np.arange(n), 64, -1)


@pytest.mark.parametrize("R", [1, 2, 3, 7, 15, 16, 17, 63, 200, 1000, 4096])
def test_windows(R):
    n = 16999
    wl = near_dag(n, 2, min(R + 20, 400), 6)  # more than four near successors: count tables
    check(wl, np.arange(n), R, -1)


@pytest.mark.parametrize("frac", [4000, 300, 20])
def test_memory_caps(frac):
    """Caps of a few to a hundred nodes, single nodes above the cap among them."""
    n = 40000
    wl = near_dag(n, 3, 60, 3)
    check(wl, np.arange(n), 100, max(1, int(wl.mem.sum()) // frac // 10))
    check(wl, np.arange(n), 100, int(np.percentile(wl.mem, 80)))


def test_wide_windows_three_targets():
    """262,145 nodes and more with R = 3,000 (three targets per lane) and 4,096
    (the staged window leaves room for one)."""
    wl = graphs._layered_config(5, 3, 330, 800, 3, 4)
    lev, oid, lp, L = O.topo_levels(wl)
    for R in (3000, 4096):
        check(wl, oid, R, -1, policy=False)


def test_many_count_tables():
    """A tile with more positions of many near successors than its LDS holds
    tables for (R = 1,000, three targets per lane: the rest from global
    memory), and tables of counts past 16 bits (parallel edges)."""
    n = 263000
    rng = np.random.default_rng(8)
    hub = rng.choice(n - 1100, 30000, replace=False)
    src = np.concatenate([np.repeat(hub, 6), np.arange(n - 1)])
    dst = src + np.concatenate([rng.integers(1, 1000, hub.size * 6), np.ones(n - 1, np.int64)])
    wl = from_edges(n, np.stack([src, dst], 1), rng.integers(0, 50, n), rng.integers(0, 3000, n), 2, [10 ** 12] * 2,
                    7, 3)
    check(wl, np.arange(n), 1000, 10 ** 12)
    n = 5000
    src = np.concatenate([np.full(70000, 700), np.full(3000, 701), np.arange(n - 1)])
    dst = np.concatenate([rng.integers(701, 760, 70000), rng.integers(702, 800, 3000), np.arange(1, n)])
    wl = from_edges(n, np.stack([src, dst], 1), rng.integers(0, 50, n), rng.integers(0, 300, n), 2, [10 ** 12] * 2, 7, 3)
    check(wl, np.arange(n), 90, 10 ** 12)


@pytest.mark.parametrize("n", [16384, 70001])
def test_workgroups_kept_off_the_gpu(n):
    """The iteration's barriers give up (forced from the host: every workgroup
    ends at its first wait): the blocked DP gives the result."""
    wl = near_dag(n, 5, 90, 3)
    was = cel.policy_iteration(3)
    try:
        check(wl, np.arange(n), 64, -1, policy=False)
        assert cel.cluster_info() == (1, 0)
    finally:
        cel.policy_iteration(was)
    check(wl, np.arange(n), 64, -1)
