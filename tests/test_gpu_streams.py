"""Calls on one device from several host threads, each on its own stream: the
kernels that spread over the whole GPU and wait for each other's workgroups
take turns, and every call gives the oracle's results."""
from __future__ import annotations

import threading
import time

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


def test_call_without_a_turn():
    """A call whose stream is behind a caller's long kernel holds the turn; one
    on another stream waits a second for it, then takes the blocked DP."""
    wl = near_dag(16384, 4)
    ref = O.cluster(wl, np.arange(wl.n), 64, -1)
    g, d = cel.Graph.from_arrays(wl, DEV), cel.Devices.from_arrays(wl)
    order = torch.arange(wl.n, dtype=torch.int32, device=DEV)
    cel.cluster(g, d, order, 64, -1)
    ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
    ev[0].record()
    torch.cuda._sleep(1 << 24)
    ev[1].record()
    torch.cuda.synchronize()
    cycles = int((1 << 24) * 2500.0 / max(ev[0].elapsed_time(ev[1]), 1e-3))  # 2.5 s
    errors, queued = [], threading.Event()

    def holder():
        try:
            s = torch.cuda.Stream()
            with torch.cuda.stream(s):
                torch.cuda._sleep(cycles)
                queued.set()
                lev, _, _, L = cel.topo_levels(g)  # takes the turn, then waits for the kernel before it
                assert L == O.topo_levels(wl)[3] and cel.topo_levels_info()[0] == 0
        except BaseException as e:  # noqa: BLE001 (reported by the test's thread)
            errors.append(repr(e))

    t = threading.Thread(target=holder)
    t.start()
    queued.wait()
    time.sleep(0.3)
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        t0 = time.perf_counter()
        cid, C, cut = cel.cluster(g, d, order, 64, -1)
        waited = time.perf_counter() - t0
    info = cel.cluster_info()
    t.join()
    print(f"[turn] waited {waited:.2f} s, {info}", flush=True)
    assert not errors, errors
    assert (C, cut) == (ref[1], ref[2]) and np.array_equal(cid.cpu().numpy(), ref[0])
    assert info == (1, 0) and 0.9 < waited < 1.3
