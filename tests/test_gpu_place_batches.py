"""GPU parity of Adjusting Placement's batched kernel (up to 64 devices) against
the CPU oracle, tolerance 0: cluster counts around its batches of 15, in-edges
from the same batch, the two before and far back, device counts around the
lane groups, busy lists that outgrow their LDS share, and co-location
followers whose leading cluster is near or far."""
from __future__ import annotations

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # collected on CPU, skipped there
    pytest.skip("needs a ROCm GPU", allow_module_level=True)

import paper_2208_00184_amd as cel  # noqa: E402
from oracle import oracle as O  # noqa: E402
from workloads import from_edges  # noqa: E402

DEV = "cuda:0"


def np_(t):
    return t.detach().cpu().numpy()


def tt(a, dt):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=dt)).to(DEV)


def clusters(n, D, seed, far, w_max, lat):
    """n clusters of one node each: in-edges from the last 31 clusters and,
    with `far`, from any; costs that leave idle gaps."""
    rng = np.random.default_rng([seed, n, D])
    edges = set()
    for v in range(1, n):
        for _ in range(int(rng.integers(0, 4))):
            edges.add((max(0, v - int(rng.integers(1, 32))), v))
        if far and v > 40:
            for u in rng.integers(0, v, int(rng.integers(0, 4))):
                edges.add((int(u), v))
    if far and n > 120:  # one cluster with more than 64 far and near in-edges
        edges |= {(u, n - 1) for u in range(0, n - 1, 1 if n < 400 else 3)}
    w = rng.integers(0, w_max, n)
    ob = rng.integers(0, 400, n)
    mem = rng.integers(1, 100, n)
    cap = [max(1, int(mem.sum()) * int(rng.integers(8, 20)) // (10 * D))] * D
    return from_edges(n, sorted(edges), w, ob, D, cap, 7, lat, mem=mem)


def check(wl, het=None, grp=None, G=0, ext=False):
    n = wl.n
    cid = np.arange(n, dtype=np.int32)
    g, d = cel.Graph.from_arrays(wl, DEV), cel.Devices.from_arrays(wl)
    if not ext:
        ref = O.place(wl, cid, n, want_fin=True)
        cdev, _, span, be, fin = cel.place(g, d, tt(cid, np.int32), n, want_fin=True)
    else:
        ref = O.place_ext(wl, cid, n, group=grp, n_groups=G, **(het or {}))
        cdev, ndev, span, be, fin = cel.place_ext(
            g, d, tt(cid, np.int32), n, group=None if grp is None else tt(grp, np.int32), n_groups=G, **(het or {}))
        assert np.array_equal(np_(ndev), ref[1])
    assert span == ref[2] and be == ref[3]
    assert np.array_equal(np_(cdev), ref[0]) and np.array_equal(np_(fin), ref[4])


@pytest.mark.parametrize("n", [1, 2, 14, 15, 16, 29, 30, 31, 45, 46, 61, 500])
def test_batch_edges(n):
    for far in (False, True):
        check(clusters(n, 3, 1, far, 60, 20))


@pytest.mark.parametrize("D", [1, 2, 15, 16, 17, 32, 33, 63, 64])
def test_device_counts(D):
    for seed, (w_max, lat) in enumerate(((60, 20), (3, 0), (2000, 1))):
        check(clusters(300, D, seed, True, w_max, lat))


def test_busy_lists_outgrow_lds():
    """64 devices share the lists' LDS: 48 blocks each (16 with the extended
    form's tables); chains of short clusters behind slow transfers leave more."""
    rng = np.random.default_rng(5)
    n, D = 6000, 64
    edges = [(v - int(rng.integers(1, 28)), v) for v in range(28, n)]
    w = rng.integers(1, 6, n)
    wl = from_edges(n, edges, w, rng.integers(0, 30, n), D, [10 ** 9] * D, 7, 3, mem=np.ones(n, np.int64))
    check(wl)
    check(wl, het=dict(tmul=[1024 + 512 * (x % 3) for x in range(D)]), ext=True)


def hetero(D, rng):
    return dict(tmul=[int(rng.integers(512, 4096)) for _ in range(D)],
                bw=[[int(rng.integers(1, 40)) for _ in range(D)] for _ in range(D)],
                lat=[[int(rng.integers(0, 50)) for _ in range(D)] for _ in range(D)])


@pytest.mark.parametrize("n,D", [(1, 1), (15, 2), (31, 5), (46, 16), (400, 17), (300, 64)])
def test_extended(n, D):
    rng = np.random.default_rng([n, D])
    wl = clusters(n, D, 7, True, 60, 20)
    het = hetero(D, rng)
    G = max(1, n // 6)  # groups over half the clusters: leaders near and far
    grp = np.where(rng.random(n) < 0.5, rng.integers(0, G, n), -1).astype(np.int32)
    near = np.where(np.arange(n) % 3 == 0, np.arange(n) // 12, -1).astype(np.int32)
    check(wl, ext=True)
    check(wl, het=het, ext=True)
    check(wl, het=dict(tmul=het["tmul"]), grp=grp, G=G, ext=True)
    check(wl, het=het, grp=grp, G=G, ext=True)
    check(wl, het=dict(bw=het["bw"]), grp=near, G=n // 12 + 1, ext=True)


def test_extended_large_transfers():
    """Summed output bytes above 2^51 on a link take the integer division."""
    n, D = 60, 4
    rng = np.random.default_rng(3)
    edges = [(v - 1 - int(rng.integers(0, min(v, 20))), v) for v in range(1, n)]
    ob = rng.integers(1 << 50, 1 << 54, n)
    wl = from_edges(n, edges, rng.integers(0, 1 << 30, n), ob, D, [10 ** 6] * D, 1 << 20, 3,
                    mem=rng.integers(1, 10, n))
    bw = [[int(rng.integers(1 << 10, 1 << 30)) for _ in range(D)] for _ in range(D)]
    check(wl, het=dict(bw=bw), ext=True)
