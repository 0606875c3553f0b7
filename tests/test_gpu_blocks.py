"""GPU parity of the makespans taken in blocks of tasks in LDS (the device
models without insertion; batches of placements over narrow levels) against the CPU oracle, tolerance 0: task counts around the blocks of 2,048, rows of
more than four and sixteen inputs in and before the block, blocks whose listed
inputs do not fit (taken again at half the size), long chains of one device,
every model with and without heterogeneous devices, and values past the packed
words, which take the other method."""
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


def tt(a, dt):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=dt)).to(DEV)


def dag(n, D, seed, fan=3, reach=300, ob_max=400, w_max=60, hubs=()):
    """In-edges from up to `reach` nodes back (every tenth node from anywhere);
    hubs: (node, in-edges) pairs."""
    rng = np.random.default_rng([seed, n, D])
    k = rng.integers(0, fan + 1, n)
    k[0] = 0
    dst = np.repeat(np.arange(n), k)
    back = np.where(dst % 10 == 0, dst, np.minimum(dst, reach))
    src = dst - 1 - (rng.random(dst.size) * back).astype(np.int64)
    e = [np.stack([src, dst], 1)]
    for v, c in hubs:
        e.append(np.stack([rng.integers(0, v, c), np.full(c, v)], 1))
    e = np.concatenate(e)
    return from_edges(n, e[e[:, 0] < e[:, 1]], rng.integers(0, w_max, n), rng.integers(0, ob_max, n), D,
                      [10 ** 15] * D, 7, 3)


def placements(n, D, K, seed):
    """Runs on one device, as clusters leave them, and scattered nodes."""
    rng = np.random.default_rng([seed, n, D, 5])
    P = np.empty((K, n), np.uint8)
    for k in range(K):
        run = max(1, [1, 40, 700, n][k % 4])
        P[k] = np.repeat(rng.integers(0, D, n // run + 1), run)[:n]
    return P


def took_blocks(yes):
    path, its, blocks = cel.makespan_blocks_info()
    print(f"[blocks] path {path}, {its} iterations, {blocks} blocks", flush=True)
    assert yes is None or path == (0 if yes else 1)
    return its, blocks


def check_model(wl, P, model, blocks=True, **het):
    g, d = cel.Graph.from_arrays(wl, DEV), cel.Devices.from_arrays(wl)
    order = np.arange(wl.n)
    ms, st, fi = cel.makespan_model(g, d, tt(order, np.int32), tt(P, np.uint8), model, want_times=True, **het)
    rm, rs, rf = O.makespan_model(wl, order, P, model, **het)
    assert np.array_equal(ms.cpu().numpy(), rm), model
    assert np.array_equal(fi.cpu().numpy(), rf) and np.array_equal(st.cpu().numpy(), rs), model
    return took_blocks(blocks)


def hetero(D, seed):
    rng = np.random.default_rng([seed, D])
    return dict(tmul=[int(x) for x in rng.integers(512, 4096, D)], bw=rng.integers(1, 40, (D, D)).tolist(),
                lat=rng.integers(0, 50, (D, D)).tolist())


@pytest.mark.parametrize("n", [1024, 2047, 2049, 4097, 9000])
@pytest.mark.parametrize("model", [0, cel.MODEL_COMM_TASKS, cel.MODEL_COMM_BLOCK])
def test_models(n, model):
    """FIFO devices take the blocks from 4,096 nodes on, transfers from 1,024."""
    for D in (2, 16, 64):
        P = placements(n, D, 4, 3)
        check_model(dag(n, D, 3), P, model, blocks=model != 0 or n >= 4096)
        check_model(dag(n, D, 3), P[:2], model, blocks=model != 0 or n >= 4096, **hetero(D, 4))


def test_one_device_and_tmul_only():
    for model in (0, cel.MODEL_COMM_TASKS, cel.MODEL_COMM_BLOCK):
        check_model(dag(4500, 1, 5), placements(4500, 1, 1, 5), model)
        check_model(dag(4500, 3, 5), placements(4500, 3, 2, 5), model, tmul=[1024, 2048, 700])


def test_long_rows():
    """Rows of 5 to 40 inputs everywhere, and hubs of hundreds and thousands."""
    wl = dag(9000, 6, 6, fan=40, reach=90, hubs=((4000, 3000), (4100, 70), (8191, 9000), (8995, 200)))
    P = placements(9000, 6, 4, 6)
    for model in (0, cel.MODEL_COMM_TASKS, cel.MODEL_COMM_BLOCK):
        check_model(wl, P[:2], model)
        check_model(wl, P[:1], model, **hetero(6, 7))


def test_listed_inputs_do_not_fit():
    """A node of 20,000 parallel in-edges from its block: blocks are halved
    until few of its sources are beside it, and grow again behind it."""
    wl = dag(4500, 3, 8)
    rng = np.random.default_rng(9)
    src = np.concatenate([np.repeat(np.arange(wl.n), np.diff(wl.out_ptr)), rng.integers(3000, 3090, 20000)])
    dst = np.concatenate([wl.out_idx, np.full(20000, 3100)])
    wl = from_edges(wl.n, np.stack([src, dst], 1), wl.w, wl.ob, 3, [10 ** 15] * 3, 7, 3)
    P = placements(4500, 3, 3, 8)
    for model in (0, cel.MODEL_COMM_TASKS, cel.MODEL_COMM_BLOCK):
        its, blocks = check_model(wl, P[:2], model)
        assert blocks <= 24  # 3 chunks of nodes alone, 5 with transfers


def test_budget_spent_on_small_blocks():
    """Forty nodes of 20,000 parallel in-edges each: small blocks one after the
    other spend the budget of iterations (64 + 0.035 n), and the call stops
    there and walks."""
    wl = dag(4500, 3, 18)
    rng = np.random.default_rng(19)
    hub = 200 + 100 * np.arange(40)
    src = np.concatenate([np.repeat(np.arange(wl.n), np.diff(wl.out_ptr))] + [rng.integers(h - 90, h, 20000) for h in hub])
    dst = np.concatenate([wl.out_idx, np.repeat(hub, 20000)])
    wl = from_edges(wl.n, np.stack([src, dst], 1), wl.w, wl.ob, 3, [10 ** 15] * 3, 7, 3)
    its, blocks = check_model(wl, placements(4500, 3, 2, 18), 0, blocks=False)
    assert 221 < its <= 260 and blocks > 20


def test_rows_longer_than_the_list():
    """Nodes fed by every node before them, 17,000 to 19,999 inputs, two in one
    block: only the inputs beside them are listed, so no block is halved."""
    n = 20000
    wl = dag(n, 6, 17, reach=60)
    e = [np.stack([np.repeat(np.arange(n), np.diff(wl.out_ptr)), wl.out_idx], 1)]
    e += [np.stack([np.arange(v), np.full(v, v)], 1) for v in (17000, 17100, n - 1)]
    wl = from_edges(n, np.concatenate(e), wl.w, wl.ob, 6, [10 ** 15] * 6, 7, 3)
    P = placements(n, 6, 4, 17)
    for model in (0, cel.MODEL_COMM_TASKS, cel.MODEL_COMM_BLOCK):
        its, blocks = check_model(wl, P[:2], model)
        assert blocks <= (10 if model == 0 else 60)  # tasks: a transfer for every device a node feeds
    its, blocks = check_model(wl, P[:1], 0, **hetero(6, 7))
    assert blocks == 10
    check_batch(wl, P)
    assert cel.makespan_blocks_info()[2] == 10


def test_values_past_the_packed_words():
    wl = dag(2500, 4, 10, ob_max=1 << 40, w_max=1 << 45)
    P = placements(2500, 4, 3, 10)
    for model in (0, cel.MODEL_COMM_TASKS, cel.MODEL_COMM_BLOCK):
        check_model(wl, P[:2], model, blocks=False)
        check_model(wl, P[:1], model, blocks=False, **hetero(4, 11))


def test_alternating_channels():
    """A chain that hops between two devices: every transfer waits for the
    last, whatever the policy starts from."""
    n = 5000
    wl = from_edges(n, [(v, v + 1) for v in range(n - 1)], np.ones(n, np.int64), np.full(n, 50), 2, [10 ** 9] * 2, 7, 3)
    P = (np.arange(n) % 2).astype(np.uint8)[None, :]
    for model in (0, cel.MODEL_COMM_TASKS, cel.MODEL_COMM_BLOCK):
        check_model(wl, P, model)


def check_batch(wl, P, seed=0, blocks=True):
    """cel.makespan of a batch, with and without its own allocations, in level
    order with the ids shuffled inside each level."""
    lev, _, lp, L = O.topo_levels(wl)
    order = np.lexsort((np.random.default_rng(seed).permutation(wl.n), lev)).astype(np.int32)
    g, d = cel.Graph.from_arrays(wl, DEV), cel.Devices.from_arrays(wl)
    args = (tt(order, np.int32), tt(lev, np.int32), tt(lp, np.int32), L, tt(P, np.uint8))
    rm, rs, rf = O.makespan(wl, order, P)
    for fixed in (False, True):
        ms, st, fi = cel.makespan(g, d, *args, want_times=True, noalloc=fixed)
        assert np.array_equal(ms.cpu().numpy(), rm), (wl.n, L, fixed)
        took_blocks(blocks)
        assert np.array_equal(fi.cpu().numpy(), rf) and np.array_equal(st.cpu().numpy(), rs), (wl.n, L, fixed)
        ms, st, fi = cel.makespan(g, d, *args, noalloc=fixed)
        assert np.array_equal(ms.cpu().numpy(), rm) and st is None and fi is None
    return L


@pytest.mark.parametrize("n", [1023, 1024, 1025, 2047, 2048, 2049, 4097, 9000])
@pytest.mark.parametrize("D", [1, 2, 16, 64, 65, 255])
def test_batches_of_placements(n, D):
    L = check_batch(dag(n, D, 12, reach=60), placements(n, D, 5, 12), n, blocks=n >= 1024)
    assert n <= 48 * L  # narrow enough for the blocks (from 1,024 nodes on)


@pytest.mark.parametrize("K,width,blocks", [(6, 47, True), (32, 48, True), (6, 49, False), (33, 40, True),
                                            (33, 41, False)])
def test_batches_by_level_width(K, width, blocks):
    """Full levels of one width, each node fed by two of the level before;
    batches of more than 32 leave the blocks at a smaller width."""
    n = 40 * width
    v = np.arange(width, n)
    rng = np.random.default_rng(width)
    e = np.concatenate([np.stack([(v // width - 1) * width + rng.integers(0, width, v.size), v], 1) for _ in range(2)])
    wl = from_edges(n, e, rng.integers(0, 60, n), rng.integers(0, 400, n), 8, [10 ** 15] * 8, 7, 3)
    assert check_batch(wl, placements(n, 8, K, 13), blocks=blocks) == 40


def test_batches_at_the_limits():
    """Values past the packed words (the ring runs); hubs whose inputs do not
    fit beside their block; more scattered placements than CUs."""
    check_batch(dag(2500, 4, 14, ob_max=1 << 40, w_max=1 << 45, reach=60), placements(2500, 4, 4, 14), blocks=False)
    check_batch(dag(9000, 6, 15, fan=40, reach=90, hubs=((4000, 3000), (8191, 17000))), placements(9000, 6, 4, 15))
    n, rng = 3000, np.random.default_rng(16)
    L = check_batch(dag(n, 3, 16, reach=20, ob_max=4000, w_max=3), rng.integers(0, 3, (300, n)).astype(np.uint8))
    assert n <= 40 * L
