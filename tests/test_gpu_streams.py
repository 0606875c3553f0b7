"""Calls on one device from several host threads, each on its own stream: the
kernels that spread over the whole GPU and wait for each other's workgroups
take turns, and every call gives the oracle's results."""
from __future__ import annotations

import threading

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # collected on CPU, skipped there
    pytest.skip("needs a ROCm GPU", allow_module_level=True)

import paper_2208_00184_amd as cel  # noqa: E402
from oracle import oracle as O  # noqa: E402
from workloads import from_edges, make_config  # noqa: E402

DEV = "cuda:0"


def near_dag(n, seed):
    rng = np.random.default_rng([seed, n])
    src = np.repeat(np.arange(n - 1), rng.integers(0, 4, n - 1))
    dst = np.minimum(n - 1, src + rng.integers(1, 91, src.size))
    ob = rng.integers(0, 3000, n)
    return from_edges(n, np.stack([src, dst], 1), rng.integers(0, 50, n), ob, 4, [int(2 * ob.sum()) + 1] * 4, 7, 3)


def oracle_plan(wl, R):
    lev, oid, lp, L = O.topo_levels(wl)
    bl, tl, prio, cp = O.blevel(wl, lev, oid)
    cid, C, cut = O.cluster(wl, prio, R, -1)
    dev = (np.arange(wl.n) * 4 // wl.n).astype(np.uint8)[None, :]
    return dict(lev=lev, oid=oid, bl=bl, tl=tl, prio=prio, cid=cid, cut=cut, dev=dev, ms=O.makespan(wl, prio, dev)[0])


def plan(g, d, R, ref, rounds, errors, go):
    try:
        s = torch.cuda.Stream()
        with torch.cuda.stream(s):
            go.wait()
            for _ in range(rounds):
                lev, oid, lp, L = cel.topo_levels(g)
                bl, tl, prio, _ = cel.blevel(g, d, lev, lp, oid, L, want_tlevel=True)
                cid, _, cut = cel.cluster(g, d, prio, R, -1)
                dev = torch.from_numpy(ref["dev"]).to(DEV)
                ms, _, _ = cel.makespan(g, d, prio, lev, lp, L, dev)
                got = dict(lev=lev, oid=oid, bl=bl, tl=tl, prio=prio, cid=cid, ms=ms)
                assert cut == ref["cut"]
                for k, v in got.items():
                    assert np.array_equal(v.cpu().numpy(), ref[k]), k
    except BaseException as e:  # noqa: BLE001 (reported by the test's thread)
        errors.append(repr(e))


def test_plans_on_four_streams():
    """Clustering of 16,384 nodes spreads over 256 workgroups of a whole CU
    each; levels, b-level, t-level and makespan over one a 1,024 nodes."""
    wls = [near_dag(16384, 1), near_dag(20011, 2), near_dag(3072, 3), make_config(3, 0)]
    refs = [oracle_plan(wl, 64) for wl in wls]
    errors, go = [], threading.Event()
    ts = [threading.Thread(target=plan, args=(cel.Graph.from_arrays(wl, DEV), cel.Devices.from_arrays(wl), 64, ref, 6,
                                              errors, go)) for wl, ref in zip(wls, refs)]
    torch.cuda.synchronize()
    for t in ts:
        t.start()
    go.set()
    for t in ts:
        t.join()
    assert not errors, errors
