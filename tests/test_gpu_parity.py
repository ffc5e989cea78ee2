"""GPU parity: every stage of the HIP library against the CPU oracle on the same seeded inputs,
called through the C ABI (paper_2109_01838_amd.binding -> librama_hip.so).

Stage-wise tests hand each GPU stage the oracle's input for that stage.  Integer results
(cycle lists, edge lists, contraction mappings, labels) must match bit-exactly; fp32 reduced
costs and lower bounds within 1e-4 relative; end to end the primal cost within 0.5 % and the
lower bound within 1e-4 relative.
"""
import numpy as np
import pytest

from paper_2109_01838_amd import inputs

pytestmark = pytest.mark.gpu

REL = 1e-4


@pytest.fixture(scope="module")
def rama():
    from paper_2109_01838_amd import Rama
    r = Rama("cuda:0")
    yield r
    r.close()


def np_(t):
    return t.detach().cpu().numpy()


def signed(g, seed, pos=0.7):
    rng = np.random.default_rng(seed)
    c = np.where(rng.random(g["c"].size) < pos, np.abs(g["c"]), -np.abs(g["c"])).astype(np.float32)
    return dict(g, c=c)


def cases():
    """name -> instance; sizes span several sort tiles (5120 or 6144 keys), on both sides of the 32-tile switch between the two offset schemes, and several 2048-item scan tiles, with ragged tails."""
    out = {}
    out["cfg1"] = inputs.cfg1()
    out["grid2d_longrange_96"] = inputs.cfg2(h=96, w=96, n_seeds=20)
    out["knn_20000"] = inputs.cfg3(n_points=20000, n_seeds=100)
    out["grid3d_24"] = inputs.cfg5_crop(24)
    out["random_dense"] = signed(inputs.random_graph(300, 6000, 11), 11, 0.6)
    out["random_sparse"] = signed(inputs.random_graph(5000, 14000, 12), 12, 0.8)
    out["messy"] = inputs.random_graph(200, 3000, 13, allow_messy=True)
    return out


CASES = cases()


def rel_close(a, b, rel=REL):
    a, b = np.asarray(a, np.float64), np.asarray(b, np.float64)
    scale = max(1.0, float(np.abs(b).max()) if b.size else 1.0)
    return np.all(np.abs(a - b) <= rel * scale)


# --------------------------------------------------------------------------------------------
# a1 cycles
# --------------------------------------------------------------------------------------------
@pytest.fixture
def search_mode(rama, request):
    """The ways of finding the cycles of length 4 and more: 1 = the per-thread walk that fetches a row per path
    at its last level, 3 = the walk whose last level closes from the far endpoint's side, 2 = the hashed
    search for lengths 4 and 5 (edges whose rows fit no table fall back to walk 3 one by one)."""
    rama.set_cycle_search(request.param)
    yield request.param
    rama.set_cycle_search(0)


BOTH_SEARCHES = pytest.mark.parametrize("search_mode", [1, 2, 3], indirect=True, ids=["walk", "hashed", "walk-meet"])


@pytest.mark.parametrize("name", list(CASES))
@pytest.mark.parametrize("lmax", [3, 4, 5])
@BOTH_SEARCHES
def test_cycles_bit_exact(rama, oracle32, name, lmax, search_mode):
    g = CASES[name]
    if name == "random_dense" and lmax == 5:
        g = dict(g, i=g["i"][:2500], j=g["j"][:2500], c=g["c"][:2500])
    want = oracle32.find_conflicted_cycles(g["n_nodes"], g["i"], g["j"], g["c"], lmax)
    got = rama.find_conflicted_cycles(g["n_nodes"], g["i"], g["j"], g["c"], lmax)
    assert len(got) == len(want) == lmax - 2
    for L in range(lmax - 2):
        assert np.array_equal(np_(got[L]), want[L]), (name, lmax, L + 3, got[L].shape, want[L].shape)


def fan_graph(d_a, d_b, row, isolated, seed=0):
    """One repulsive edge (0, last) between a node with d_a and a node with d_b attractive neighbours, three of them
    shared; every neighbour has `row` more attractive neighbours among 300 middle nodes, some of which are the other
    side's neighbours.  `isolated` further nodes bring the average row down."""
    rng = np.random.default_rng(seed)
    side_a = np.arange(1, 1 + d_a)
    side_b = np.concatenate([side_a[:3], np.arange(1 + d_a, 1 + d_a + d_b)])[:d_b]
    last = 1 + d_a + d_b + 300 + isolated
    middle = np.arange(1 + d_a + d_b, 301 + d_a + d_b)
    edges = [(0, x) for x in side_a] + [(x, last) for x in side_b]
    for x in np.unique(np.concatenate([side_a, side_b])):
        edges += [(x, y) for y in rng.choice(middle, row, replace=False)]
    edges += [(x, y) for x in side_a[:5] for y in side_b[-5:] if x != y]
    key = np.unique([min(e) * (last + 1) + max(e) for e in edges])
    i = np.concatenate([key // (last + 1), [0]]).astype(np.int32)
    j = np.concatenate([key % (last + 1), [last]]).astype(np.int32)
    c = np.concatenate([1.0 + rng.random(key.size), [-1.0]]).astype(np.float32)
    return int(last + 1), i, j, c


# the limits of the hashed search: 16 lanes take rows of 16 and 15 entries and a table of 224, 64 lanes rows of 64 and
# 63 and tables of 896 and 3584 entries (entries: the rows of the far endpoint's neighbours); the next size up goes to
# the larger table or to the wave-per-edge walk
@pytest.mark.parametrize("isolated", [0, 4000], ids=["wide", "narrow"])
@pytest.mark.parametrize("d_a,d_b,row", [(1, 1, 1), (16, 15, 13), (16, 15, 14), (17, 15, 5), (16, 16, 5), (64, 63, 11), (64, 63, 14),
                                         (64, 63, 55), (64, 63, 60), (65, 63, 9), (64, 64, 9), (130, 70, 9)])
@pytest.mark.parametrize("lmax,shortest", [(4, False), (5, False), (5, True)])
def test_hashed_search_at_its_limits(rama, oracle32, isolated, d_a, d_b, row, lmax, shortest):
    n, i, j, c = fan_graph(d_a, d_b, row, isolated)
    want = oracle32.find_conflicted_cycles(n, i, j, c, lmax, shortest_only=shortest)
    rama.set_cycle_search(2)
    try:
        got = rama.find_conflicted_cycles(n, i, j, c, lmax, shortest_only=shortest)
    finally:
        rama.set_cycle_search(0)
    for L in range(lmax - 2):
        assert np.array_equal(np_(got[L]), want[L]), (L + 3, got[L].shape, want[L].shape)


# common neighbours of a repulsive edge around the sixteen there is room for between counting and writing
@pytest.mark.parametrize("pages", [0, 1, 15, 16, 17, 31, 32, 33, 200])
def test_common_neighbours_with_and_without_room(rama, oracle32, pages):
    sizes = [pages, 3, 16, 17, pages + 1]
    i, j, c, n = [], [], [], 0
    rng = np.random.default_rng(pages)
    for k in sizes:
        a, b, page = n, n + 1, n + 2 + np.arange(k)
        i += [[a], np.full(k, a), np.full(k, b)]
        j += [[b], page, page]
        c += [[-1.0], 0.5 + rng.random(k), 0.5 + rng.random(k)]
        n += k + 2
    i, j = np.concatenate(i).astype(np.int32), np.concatenate(j).astype(np.int32)
    c = np.concatenate(c).astype(np.float32)
    want = oracle32.find_conflicted_cycles(n, i, j, c, 3)
    rama.set_cycle_search(2)
    try:
        got = rama.find_conflicted_cycles(n, i, j, c, 3)
    finally:
        rama.set_cycle_search(0)
    assert np.array_equal(np_(got[0]), want[0]) and want[0].shape[0] == sum(sizes)


# items of a repulsive edge around the 64 that sixteen lanes take at a time, and the 256 of 64 lanes
@pytest.mark.parametrize("isolated", [0, 4000], ids=["wide", "narrow"])
@pytest.mark.parametrize("d_a,d_b,row", [(3, 3, 1), (7, 9, 6), (8, 8, 6), (8, 8, 7), (13, 9, 5), (16, 7, 8), (5, 13, 9), (20, 20, 11), (17, 16, 14), (30, 25, 9)])
@pytest.mark.parametrize("lmax", [4, 5])
def test_hashed_search_takes_items_in_batches(rama, oracle32, isolated, d_a, d_b, row, lmax):
    for seed in range(3):
        n, i, j, c = fan_graph(d_a, d_b, row, isolated, seed)
        want = oracle32.find_conflicted_cycles(n, i, j, c, lmax)
        got = rama.find_conflicted_cycles(n, i, j, c, lmax)
        for w, g in zip(want, got):
            assert np.array_equal(np_(g), w)


# repulsive edges without room in the tables: 4096 and more of those with up to 8 attractive neighbours at their first
# endpoint are walked by a thread each, fewer of them and those with more neighbours there by a wave each
@pytest.mark.parametrize("n_edges,row", [(4095, 8), (4096, 8), (4097, 1), (4500, 9), (9000, 4)])
@pytest.mark.parametrize("lmax,shortest", [(4, False), (5, False), (5, True)])
def test_edges_without_room_in_the_tables(rama, oracle32, n_edges, row, lmax, shortest):
    rng = np.random.default_rng(n_edges + row)
    middle = n_edges + np.arange(200)
    side = n_edges + 200 + np.arange(64)            # one entry more than a mask holds
    last = n_edges + 264
    e = [(v, x) for v in range(n_edges) for x in rng.choice(middle[: 40 * row], row, replace=False)]
    e += [(x, last) for x in side] + [(y, x) for x in side for y in rng.choice(middle, 3, replace=False)]
    e += [tuple(rng.choice(middle, 2, replace=False)) for _ in range(300)]
    key = np.unique([min(a, b) * (last + 1) + max(a, b) for a, b in e])
    i = np.concatenate([key // (last + 1), np.arange(n_edges)]).astype(np.int32)
    j = np.concatenate([key % (last + 1), np.full(n_edges, last)]).astype(np.int32)
    c = np.where(np.arange(i.size) < key.size, 1.0, -1.0).astype(np.float32)
    n = int(last) + 1
    want = oracle32.find_conflicted_cycles(n, i, j, c, lmax, shortest_only=shortest)
    assert want[1].shape[0] > 0
    got = rama.find_conflicted_cycles(n, i, j, c, lmax, shortest_only=shortest)
    for L in range(lmax - 2):
        assert np.array_equal(np_(got[L]), want[L]), (L + 3, got[L].shape, want[L].shape)


def test_search_on_a_star_is_no_slower_than_the_walk(rama):
    """Repulsive edges between the leaves of a star: every row of their far endpoints is the hub's, which no table holds.
    A wave per edge took 60 times as long as the walk with a thread per edge (2.6 s)."""
    import time
    import torch
    n = 40000
    rng = np.random.default_rng(3)
    a, b = np.sort(rng.integers(1, n, (2, 60000)), axis=0)
    a, b = a[a < b], b[a < b]
    i = torch.as_tensor(np.concatenate([np.zeros(n - 1), a]).astype(np.int32)).cuda()
    j = torch.as_tensor(np.concatenate([np.arange(1, n), b]).astype(np.int32)).cuda()
    c = torch.as_tensor(np.concatenate([np.ones(n - 1), -np.ones(a.size)]).astype(np.float32)).cuda()
    took = {}
    try:
        for mode in (0, 3):
            rama.set_cycle_search(mode)
            for _ in range(2):
                torch.cuda.synchronize()
                t = time.perf_counter()
                got = rama.find_conflicted_cycles(n, i, j, c, 5)
                torch.cuda.synchronize()
                took[mode] = time.perf_counter() - t
            assert [g.shape[0] for g in got][1:] == [0, 0] and got[0].shape[0] > 0.9 * a.size
    finally:
        rama.set_cycle_search(0)
    assert took[0] < 3 * took[3], took


def all_pairs_around_rings(n):
    """Every pair of n nodes; the nodes a few steps apart attract each other, 14 of them per node, all others repel."""
    import torch
    i, j = (x.to(torch.int32) for x in torch.triu_indices(n, n, 1, device="cuda:0"))
    c = -torch.ones(i.numel(), device="cuda:0")
    d = j - i
    for step in (1, 30, 200, 900, 2500, 4000, 5500):
        c[(d == step) | (d == n - step)] = 1.0
    return i, j, c


# (nodes, longest cycle, repulsive edges at least): a wave (lengths 4 and 5) or sixteen lanes (triangles) for each of them would
# be more than the 2^32 threads a launch may have in one dimension
@pytest.mark.parametrize("n,lmax,least", [(11900, 4, 1 << 26), (23400, 3, 1 << 28)])
def test_search_on_more_repulsive_edges_than_one_launch_has_lanes(rama, n, lmax, least):
    """The lanes stride over the edges; the lists are those of the walk."""
    import torch
    i, j, c = all_pairs_around_rings(n)
    assert int((c < 0).sum()) > least
    got = rama.find_conflicted_cycles(n, i, j, c, lmax)
    try:
        rama.set_cycle_search(3)
        want = rama.find_conflicted_cycles(n, i, j, c, lmax)
    finally:
        rama.set_cycle_search(0)
    assert want[-1].shape[0] > 1000
    for L in range(lmax - 2):
        assert torch.equal(got[L], want[L]), (L + 3, got[L].shape, want[L].shape)


def test_dual_rounds_allocates_its_result_and_nothing_else(rama, monkeypatch):
    made = []
    empty = rama._empty
    monkeypatch.setattr(rama, "_empty", lambda n, dtype: made.append(int(n)) or empty(n, dtype))
    i, j = np.arange(50, dtype=np.int32), np.arange(1, 51, dtype=np.int32)
    got = rama.dual_rounds(51, i, j, np.ones(50, np.float32))
    assert made == [50, 50, 50] and np.array_equal(np_(got["i"]), i) and np.array_equal(np_(got["j"]), j)
    got = rama.dual_rounds(51, i[:0], j[:0], np.ones(0, np.float32))
    assert all(got[k].numel() == 0 for k in "ijc")


def test_no_room_is_asked_for_what_cannot_be_written(rama):
    """7.2e8 triangles are a list of more than 2^31 numbers: the call says so before it asks its caller for 8 GiB."""
    import ctypes as C
    import torch
    from paper_2109_01838_amd import RamaError, binding
    top, many = 240, 25000
    a, b = (x.to(torch.int32) for x in torch.triu_indices(top, top, 1, device="cuda:0"))
    i = torch.cat([a, torch.arange(top, device="cuda:0", dtype=torch.int32).repeat_interleave(many)])
    j = torch.cat([b, (top + torch.arange(many, device="cuda:0", dtype=torch.int32)).repeat(top)])
    c = torch.ones(i.numel(), device="cuda:0")
    c[: a.numel()] = -1.0
    n, want = top + many, a.numel() * many
    assert 3 * want >= 1 << 31
    asked, cnt = [], (C.c_int64 * 1)()
    room = binding.RamaRoom(binding.ROOM_FN(lambda _user, which, nbytes: asked.append((which, nbytes))), None)
    st = rama.lib.rama_find_conflicted_cycles_room(rama.ctx, n, i.numel(), i.data_ptr(), j.data_ptr(), c.data_ptr(), 3, 0, C.byref(room), cnt)
    assert (st, asked, cnt[0]) == (binding.RAMA_ERR_CAPACITY, [], want)
    # the size query of the entry point with buffers answers as before
    st = rama.lib.rama_find_conflicted_cycles(rama.ctx, n, i.numel(), i.data_ptr(), j.data_ptr(), c.data_ptr(), 3, 0, None, None, cnt)
    assert (st, cnt[0]) == (binding.RAMA_ERR_CAPACITY, want)
    with pytest.raises(RamaError) as ei:
        rama.find_conflicted_cycles(n, i, j, c, 3)
    assert ei.value.status == binding.RAMA_ERR_CAPACITY and "2^31" in str(ei.value)


# graphs whose attractive rows have exactly up to 6 entries are counted with whole rows in registers; 7 take another search
@pytest.mark.parametrize("row", [1, 5, 6, 7])
def test_cycles_on_short_rows(rama, oracle32, row):
    rng = np.random.default_rng(row)
    n = 4000
    base = np.arange(n)
    offs = [1, 2, 5, 11][: (row + 1) // 2]
    i = np.concatenate([base for _ in offs])
    j = np.concatenate([(base + d) % n for d in offs])      # a circulant graph: rows of 2 * len(offs) before the cut
    if row % 2:
        cut = j != (i + offs[-1]) % n
        i, j = np.concatenate([i[cut], np.arange(0, n, 2)]), np.concatenate([j[cut], np.arange(1, n, 2)])     # odd rows: plus a pairing
        i, j = np.concatenate([i, np.arange(3)]), np.concatenate([j, np.arange(3) + 40])
    c = np.ones(i.size, np.float32)
    if not row % 2:
        c[rng.random(i.size) < 0.1] = -1.0
    extra = rng.integers(0, n, (2, 3000))
    near = (extra[0] + rng.integers(1, 30, 3000)) % n
    i, j, c = np.concatenate([i, extra[0]]).astype(np.int32), np.concatenate([j, near]).astype(np.int32), np.concatenate([c, -3.0 * np.ones(3000)]).astype(np.float32)
    n *= 2      # nodes without edges: the longest row is only looked at when rows are short on average
    want = oracle32.find_conflicted_cycles(n, i, j, c, 5)
    got = rama.find_conflicted_cycles(n, i, j, c, 5)
    assert sum(w.shape[0] for w in want) > 0 or row == 1
    for L in range(3):
        assert np.array_equal(np_(got[L]), want[L]), (L + 3, got[L].shape, want[L].shape)


# cycles of length 6 and 7 (named as future work in Sec. 5) and the shortest-only separation; the
# cases are the ones whose plain enumeration the oracle finishes in seconds
LONG_CASES = [("cfg1", 7), ("grid3d_24", 7), ("random_sparse", 7), ("knn_20000", 7), ("knn_20000", 6),
              ("grid2d_longrange_96", 6), ("messy", 6)]


@pytest.mark.parametrize("name,lmax", LONG_CASES)
@BOTH_SEARCHES
def test_longer_cycles_bit_exact(rama, oracle32, name, lmax, search_mode):
    g = CASES[name]
    want = oracle32.find_conflicted_cycles(g["n_nodes"], g["i"], g["j"], g["c"], lmax)
    got = rama.find_conflicted_cycles(g["n_nodes"], g["i"], g["j"], g["c"], lmax)
    assert len(got) == lmax - 2
    for L in range(lmax - 2):
        assert np.array_equal(np_(got[L]), want[L]), (name, lmax, L + 3, got[L].shape, want[L].shape)
    print(name, lmax, [x.shape[0] for x in want])


@pytest.mark.parametrize("name", list(CASES))
@pytest.mark.parametrize("lmax", [3, 4, 5, 7])
@BOTH_SEARCHES
def test_shortest_only_cycles_bit_exact(rama, oracle32, name, lmax, search_mode):
    g = CASES[name]
    if name in ("random_dense", "messy") and lmax == 7:
        g = dict(g, i=g["i"][:1500], j=g["j"][:1500], c=g["c"][:1500])
    want = oracle32.find_conflicted_cycles(g["n_nodes"], g["i"], g["j"], g["c"], lmax, shortest_only=True)
    got = rama.find_conflicted_cycles(g["n_nodes"], g["i"], g["j"], g["c"], lmax, shortest_only=True)
    for L in range(lmax - 2):
        assert np.array_equal(np_(got[L]), want[L]), (name, lmax, L + 3, got[L].shape, want[L].shape)
    # every repulsive edge appears with one length only
    seen = {}
    for L, x in enumerate(np_(q) for q in got):
        for a, b in set(zip(x[:, 0].tolist(), x[:, -1].tolist())):
            assert seen.setdefault((a, b), L) == L


# skewed degrees: repulsive edges at hubs (attractive rows of ~600 entries) take the wave-per-edge path
@pytest.fixture(scope="module")
def hubs():
    return inputs.hub_graph()


@pytest.mark.parametrize("lmax,shortest", [(3, False), (4, False), (5, False), (4, True), (5, True), (7, True)])
@BOTH_SEARCHES
def test_heavy_rows_cycles_bit_exact(rama, oracle32, hubs, lmax, shortest, search_mode):
    g = hubs
    deg = np.bincount(np.concatenate([g["i"][g["c"] > 0], g["j"][g["c"] > 0]]), minlength=g["n_nodes"])
    assert deg.max() > 500 and np.median(deg) < 10
    want = oracle32.find_conflicted_cycles(g["n_nodes"], g["i"], g["j"], g["c"], lmax, shortest_only=shortest)
    got = rama.find_conflicted_cycles(g["n_nodes"], g["i"], g["j"], g["c"], lmax, shortest_only=shortest)
    for L in range(lmax - 2):
        assert np.array_equal(np_(got[L]), want[L]), (lmax, shortest, L + 3, got[L].shape, want[L].shape)
    # the hubs' own repulsive edges are among the results
    heavy = set(np.where(deg > 128)[0].tolist())
    assert any(int(v) in heavy for L in range(lmax - 2) for v in np.unique(want[L][:, 0]))
    print(lmax, shortest, [x.shape[0] for x in want])


def test_heavy_rows_solve(rama, oracle32, hubs):
    g = hubs
    n = g["n_nodes"]
    want = oracle32.solve(n, g["i"], g["j"], g["c"])
    got = rama.solve(n, g["i"], g["j"], g["c"])
    assert got["n_cycles_first"] == want["n_cycles_first"]
    assert abs(got["lower_bound"] - want["lower_bound"]) <= REL * max(1.0, abs(want["lower_bound"]))
    assert abs(got["primal"] - want["primal"]) <= 5e-3 * max(1.0, abs(want["primal"]))
    print("hubs: labels identical:", bool(np.array_equal(np_(got["labels"]), want["labels"])), got["primal"], want["primal"])


def test_cycles_capacity_protocol(rama):
    import ctypes as C
    import torch
    from paper_2109_01838_amd import binding
    g = CASES["cfg1"]
    i, j, c = (torch.as_tensor(g[k], device="cuda") for k in ("i", "j", "c"))
    cnt = (C.c_int64 * 5)()
    args = (rama.ctx, g["n_nodes"], i.numel(), i.data_ptr(), j.data_ptr(), c.data_ptr())
    st = rama.lib.rama_find_conflicted_cycles(*args, 5, 0, None, None, cnt)
    assert st == binding.RAMA_ERR_CAPACITY and cnt[1] > 0 and cnt[0] == 0 and cnt[2] == 0
    buf = torch.full((4 * (cnt[1] - 1) + 1,), -7, dtype=torch.int32, device="cuda")
    cap = (C.c_int64 * 3)(0, cnt[1] - 1, 0)
    ptrs = (C.c_void_p * 3)(None, buf.data_ptr(), None)
    st = rama.lib.rama_find_conflicted_cycles(*args, 5, 0, cap, ptrs, cnt)
    assert st == binding.RAMA_ERR_CAPACITY
    assert bool((buf == -7).all())          # nothing written on capacity failure
    cap[1] = cnt[1]
    buf = torch.full((4 * cnt[1] + 1,), -7, dtype=torch.int32, device="cuda")
    ptrs[1] = buf.data_ptr()
    st = rama.lib.rama_find_conflicted_cycles(*args, 5, 0, cap, ptrs, cnt)
    assert st == binding.RAMA_OK and int(buf[-1]) == -7 and bool((buf[:-1] >= 0).all())
    for bad_len in (2, binding.MAX_CYCLE_LEN + 1):
        st = rama.lib.rama_find_conflicted_cycles(*args, bad_len, 0, None, None, cnt)
        assert st == binding.RAMA_ERR_INVALID_ARG
    cap[1] = -1
    assert rama.lib.rama_find_conflicted_cycles(*args, 5, 0, cap, ptrs, cnt) == binding.RAMA_ERR_INVALID_ARG
    cap[1] = 5
    ptrs[1] = None
    assert rama.lib.rama_find_conflicted_cycles(*args, 5, 0, cap, ptrs, cnt) == binding.RAMA_ERR_INVALID_ARG


def test_room_for_results_of_unknown_size(rama):
    """The entry points that ask the caller for memory give what the sizing protocol gives, ask only for results that
    are not empty, and end with RAMA_ERR_OOM -- nothing written, the ctx usable -- when there is none."""
    import ctypes as C
    import torch
    from paper_2109_01838_amd import binding, default_params
    g = CASES["cfg1"]
    i, j, c = (torch.as_tensor(g[k], device="cuda") for k in ("i", "j", "c"))
    args = (rama.ctx, g["n_nodes"], i.numel(), i.data_ptr(), j.data_ptr(), c.data_ptr())
    cnt, got = (C.c_int64 * 3)(), {}

    def give(_user, which, nbytes):
        got[which] = torch.full((nbytes // 4,), -7, dtype=torch.int32, device="cuda")
        return got[which].data_ptr()

    room, none = binding.RamaRoom(binding.ROOM_FN(give), None), binding.RamaRoom(binding.ROOM_FN(lambda *_: None), None)
    assert rama.lib.rama_find_conflicted_cycles_room(*args, 5, 0, C.byref(room), cnt) == binding.RAMA_OK
    assert list(got) == [4] and cnt[0] == cnt[2] == 0
    ref = torch.full((4 * cnt[1],), -7, dtype=torch.int32, device="cuda")
    cap, ptrs = (C.c_int64 * 3)(0, cnt[1], 0), (C.c_void_p * 3)(None, ref.data_ptr(), None)
    assert rama.lib.rama_find_conflicted_cycles(*args, 5, 0, cap, ptrs, cnt) == binding.RAMA_OK
    assert torch.equal(got[4], ref)
    assert rama.lib.rama_find_conflicted_cycles_room(*args, 5, 0, C.byref(none), cnt) == binding.RAMA_ERR_OOM
    assert rama.lib.rama_find_conflicted_cycles_room(*args, 5, 0, None, cnt) == binding.RAMA_ERR_INVALID_ARG
    p, m = default_params(dual_rounds=2), C.c_int64(0)
    got.clear()
    assert rama.lib.rama_dual_rounds_room(*args, C.byref(p), C.byref(room), C.byref(m), None, None, None) == binding.RAMA_OK
    assert sorted(got) == [0, 1, 2] and all(x.numel() == m.value for x in got.values())
    ref = [torch.empty(m.value, dtype=torch.int32, device="cuda") for _ in range(3)]
    assert rama.lib.rama_dual_rounds(*args, C.byref(p), m.value - 1, *(x.data_ptr() for x in ref), C.byref(m), None, None,
                                     None) == binding.RAMA_ERR_CAPACITY
    assert rama.lib.rama_dual_rounds(*args, C.byref(p), m.value, *(x.data_ptr() for x in ref), C.byref(m), None, None,
                                     None) == binding.RAMA_OK
    assert all(torch.equal(got[q], ref[q]) for q in range(3))
    assert rama.lib.rama_dual_rounds_room(*args, C.byref(p), C.byref(none), C.byref(m), None, None, None) == binding.RAMA_ERR_OOM


# --------------------------------------------------------------------------------------------
# a2 + a3 message passing
# --------------------------------------------------------------------------------------------
@pytest.mark.parametrize("name", list(CASES))
@pytest.mark.parametrize("k", [0, 1, 10])
def test_message_passing_parity(rama, oracle32, name, k):
    g = CASES[name]
    n = g["n_nodes"]
    lmax = 4 if name == "random_dense" else 5
    cyc = oracle32.find_conflicted_cycles(n, g["i"], g["j"], g["c"], lmax)
    want = oracle32.message_passing(n, g["i"], g["j"], g["c"], cyc, k, trace=True)
    got = rama.message_passing(n, g["i"], g["j"], g["c"], cyc, k, trace=True)
    assert np.array_equal(np_(got["i"]), want["i"]) and np.array_equal(np_(got["j"]), want["j"])
    assert rel_close(np_(got["c"]), want["c"])
    assert abs(got["lower_bound"] - want["lower_bound"]) <= REL * max(1.0, abs(want["lower_bound"]))
    assert rel_close(got["lb_trace"], want["lb_trace"])
    tr = np.asarray(got["lb_trace"])
    assert np.all(np.diff(tr) >= -1e-5 * (1.0 + np.abs(tr[:-1])))       # monotone (Appendix, LB lemma)
    # the arithmetic is ordered identically on both sides, so in practice the match is exact
    print(name, k, "max |dc| =", float(np.abs(np_(got["c"]) - want["c"]).max()) if want["c"].size else 0.0,
          "bit-exact:", bool(np.array_equal(np_(got["c"]), want["c"])))


@pytest.mark.parametrize("name,lmax", LONG_CASES)
@pytest.mark.parametrize("shortest", [False, True])
def test_message_passing_parity_longer_cycles(rama, oracle32, name, lmax, shortest):
    g = CASES[name]
    n = g["n_nodes"]
    cyc = oracle32.find_conflicted_cycles(n, g["i"], g["j"], g["c"], lmax, shortest_only=shortest)
    want = oracle32.message_passing(n, g["i"], g["j"], g["c"], cyc, 5, trace=True)
    got = rama.message_passing(n, g["i"], g["j"], g["c"], cyc, 5, trace=True)
    assert np.array_equal(np_(got["i"]), want["i"]) and np.array_equal(np_(got["j"]), want["j"])
    assert rel_close(np_(got["c"]), want["c"])
    assert rel_close(got["lb_trace"], want["lb_trace"])
    print(name, lmax, shortest, "edges", want["i"].size, "bit-exact:", bool(np.array_equal(np_(got["c"]), want["c"])))


# dual rounds on one graph: the triangle set and its costs persist from round to round
DUAL_CASES = [(name, L, R) for name in CASES for (L, R) in ((3, 3), (4, 2), (5, 2))
              if not (name in ("random_dense", "messy") and L > 3) and not (name == "grid2d_longrange_96" and L == 5)]


@pytest.mark.parametrize("name,lmax,rounds", DUAL_CASES)
def test_dual_rounds_parity(rama, oracle32, name, lmax, rounds):
    from paper_2109_01838_amd import default_params
    g = CASES[name]
    n = g["n_nodes"]
    want = oracle32.dual_rounds(n, g["i"], g["j"], g["c"], lmax, 5, rounds)
    got = rama.dual_rounds(n, g["i"], g["j"], g["c"],
                           default_params(max_cycle_len_first=lmax, mp_iters_first=5, dual_rounds=rounds))
    assert np.array_equal(np_(got["i"]), want["i"]) and np.array_equal(np_(got["j"]), want["j"])
    assert rel_close(np_(got["c"]), want["c"])
    assert rel_close(got["lb_trace"], want["lb_trace"])
    assert abs(got["lower_bound"] - want["lower_bound"]) <= REL * max(1.0, abs(want["lower_bound"]))
    assert got["n_triangles"] == want["n_triangles"]
    tr = np.asarray(got["lb_trace"])
    assert np.all(np.diff(tr) >= -1e-5 * (1.0 + np.abs(tr[:-1])))
    print(name, lmax, rounds, "LB", list(tr), "triangles", got["n_triangles"], "bit-exact:",
          bool(np.array_equal(np_(got["c"]), want["c"])))


def test_dual_rounds_one_round_is_separation_plus_message_passing(rama):
    from paper_2109_01838_amd import default_params
    g = CASES["knn_20000"]
    n = g["n_nodes"]
    cyc = rama.find_conflicted_cycles(n, g["i"], g["j"], g["c"], 5)
    mp = rama.message_passing(n, g["i"], g["j"], g["c"], cyc, 10)
    one = rama.dual_rounds(n, g["i"], g["j"], g["c"], default_params(dual_rounds=1))
    assert np.array_equal(np_(one["c"]), np_(mp["c"])) and one["lower_bound"] == mp["lower_bound"]
    zero = rama.dual_rounds(n, g["i"], g["j"], g["c"], default_params(dual_rounds=0))
    assert zero["lb_trace"] == [zero["lower_bound"]] and zero["n_triangles"] == 0
    assert abs(zero["lower_bound"] - float(np.minimum(g["c"], 0).astype(np.float64).sum())) <= 1e-9 * abs(zero["lower_bound"])


def test_message_passing_cycle_order_is_irrelevant(rama, oracle32):
    g = CASES["knn_20000"]
    n = g["n_nodes"]
    cyc = oracle32.find_conflicted_cycles(n, g["i"], g["j"], g["c"], 5)
    rng = np.random.default_rng(0)
    shuffled = [x[rng.permutation(x.shape[0])] for x in cyc]
    a = rama.message_passing(n, g["i"], g["j"], g["c"], cyc, 3)
    b = rama.message_passing(n, g["i"], g["j"], g["c"], shuffled, 3)
    assert np.array_equal(np_(a["c"]), np_(b["c"])) and a["lower_bound"] == b["lower_bound"]


# chords and fan triangles of cycles of five and more nodes are made unique tile by tile (2048 candidates): lists that end on
# either side of a tile, and one in which every cycle comes twice
@pytest.mark.parametrize("n5,twice", [(1, False), (682, False), (683, False), (1023, False), (1024, False), (1025, False), (3000, True)])
@pytest.mark.parametrize("lmax", [5, 6])
def test_message_passing_repeated_chords_and_triangles(rama, oracle32, n5, twice, lmax):
    g = CASES["knn_20000"]
    n = g["n_nodes"]
    cyc = oracle32.find_conflicted_cycles(n, g["i"], g["j"], g["c"], lmax)
    cyc = [c[: n5 if q == len(cyc) - 1 else n5 // 3] for q, c in enumerate(cyc)]
    if twice:
        cyc = [np.concatenate([c, c[::-1]]) for c in cyc]
    want = oracle32.message_passing(n, g["i"], g["j"], g["c"], cyc, 3)
    got = rama.message_passing(n, g["i"], g["j"], g["c"], cyc, 3)
    assert np.array_equal(np_(got["i"]), want["i"]) and np.array_equal(np_(got["j"]), want["j"])
    assert np.array_equal(np_(got["c"]), want["c"])


def triangle_fan(hubs, n_tri, seed):
    """n_tri triangles dealt out to `hubs` repulsive edges."""
    rng = np.random.default_rng(seed)
    h, x = np.arange(n_tri) % hubs, 2 * hubs + np.arange(n_tri)
    i = np.concatenate([2 * np.arange(hubs), 2 * h, 2 * h + 1])
    j = np.concatenate([2 * np.arange(hubs) + 1, x, x])
    c = rng.uniform(0.5, 1.5, i.size)
    c[:hubs] *= -1
    order = np.lexsort((j, i))
    return 2 * hubs + n_tri, i[order].astype(np.int32), j[order].astype(np.int32), c[order].astype(np.float32)


# edges in as many triangles as are compared with each other, and in one more; as many long ones as there can be
@pytest.mark.parametrize("hubs,n_tri", [(1, 256), (1, 257), (1, 2047), (1, 2048), (1, 2049), (7, 7 * 257), (7, 2048), (8, 2048), (3, 1000)])
@pytest.mark.parametrize("k", [1, 4])
def test_message_passing_of_edges_in_many_triangles(rama, oracle32, hubs, n_tri, k):
    n, i, j, c = triangle_fan(hubs, n_tri, n_tri)
    cyc = oracle32.find_conflicted_cycles(n, i, j, c, 3)
    cyc = [x[np.random.default_rng(1).permutation(x.shape[0])] for x in cyc]
    want = oracle32.message_passing(n, i, j, c, cyc, k)
    got = rama.message_passing(n, i, j, c, cyc, k)
    assert np.array_equal(np_(got["i"]), want["i"]) and np.array_equal(np_(got["j"]), want["j"])
    assert np.array_equal(np_(got["c"]), want["c"])


def test_one_workgroup_is_no_slower_on_an_edge_in_all_triangles(rama):
    """2048 triangles are passed by one workgroup, 2049 by the kernels for any number."""
    import time
    import torch
    best = {}
    for n_tri in (2048, 2049):
        n, *g = triangle_fan(1, n_tri, 3)
        g = [torch.as_tensor(x).cuda() for x in g]
        cyc = rama.find_conflicted_cycles(n, *g, max_cycle_len=3)
        for _ in range(20):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            rama.message_passing(n, *g, cyc, 1)
            torch.cuda.synchronize()
            best[n_tri] = min(best.get(n_tri, 1.0), time.perf_counter() - t0)
    assert best[2048] <= 1.3 * best[2049], best


def test_message_passing_rejects_foreign_cycles(rama):
    from paper_2109_01838_amd import RamaError, binding
    g = CASES["cfg1"]
    bad = [np.array([[0, 1, 40]], np.int32), np.zeros((0, 4), np.int32), np.zeros((0, 5), np.int32)]
    with pytest.raises(RamaError) as ei:
        rama.message_passing(g["n_nodes"], g["i"], g["j"], g["c"], bad, 1)
    assert ei.value.status == binding.RAMA_ERR_BAD_GRAPH
    bad[0] = np.array([[0, 1, 5000]], np.int32)
    with pytest.raises(RamaError):
        rama.message_passing(g["n_nodes"], g["i"], g["j"], g["c"], bad, 1)


# --------------------------------------------------------------------------------------------
# a4-a6 contraction
# --------------------------------------------------------------------------------------------
@pytest.mark.parametrize("name", list(CASES))
@pytest.mark.parametrize("repeat", [1, 0])
def test_contract_parity(rama, oracle32, name, repeat):
    g = CASES[name]
    n = g["n_nodes"]
    # the stage input is what the oracle's dual step hands over: reduced costs incl. chords
    cyc = oracle32.find_conflicted_cycles(n, g["i"], g["j"], g["c"], 4)
    mp = oracle32.message_passing(n, g["i"], g["j"], g["c"], cyc, 5)
    want = oracle32.contract(n, mp["i"], mp["j"], mp["c"], repeat=repeat)
    got = rama.contract(n, mp["i"], mp["j"], mp["c"], repeat=repeat)
    assert got["n_nodes"] == want["n_nodes"]
    assert np.array_equal(np_(got["mapping"]), want["mapping"])
    assert np.array_equal(np_(got["i"]), want["i"]) and np.array_equal(np_(got["j"]), want["j"])
    assert rel_close(np_(got["c"]), want["c"])
    assert rel_close(np_(got["diag"]), want["diag"])
    print(name, repeat, "costs bit-exact:", bool(np.array_equal(np_(got["c"]), want["c"])),
          "diag bit-exact:", bool(np.array_equal(np_(got["diag"]), want["diag"])))


@pytest.mark.parametrize("name", list(CASES))
@pytest.mark.parametrize("repeat", [1, 0])
def test_contract_forest_parity(rama, oracle32, name, repeat):
    """forest_ratio=1 forces the spanning forest without conflicts in every primal update."""
    from paper_2109_01838_amd import default_params
    g = CASES[name]
    n = g["n_nodes"]
    cyc = oracle32.find_conflicted_cycles(n, g["i"], g["j"], g["c"], 4)
    mp = oracle32.message_passing(n, g["i"], g["j"], g["c"], cyc, 5)
    want = oracle32.contract(n, mp["i"], mp["j"], mp["c"], repeat=repeat, forest_ratio=1.0)
    got = rama.contract(n, mp["i"], mp["j"], mp["c"], params=default_params(forest_ratio=1.0), repeat=repeat)
    assert got["n_nodes"] == want["n_nodes"]
    assert np.array_equal(np_(got["mapping"]), want["mapping"])
    assert np.array_equal(np_(got["i"]), want["i"]) and np.array_equal(np_(got["j"]), want["j"])
    assert rel_close(np_(got["c"]), want["c"])
    assert rel_close(np_(got["diag"]), want["diag"])
    # no repulsive input edge ends up inside a cluster after ONE forest update
    if repeat == 1:
        mp_ = want["mapping"]
        assert not np.any((mp["c"] < 0) & (mp_[mp["i"]] == mp_[mp["j"]]))


@pytest.mark.parametrize("n", [9, 26, 30, 31, 32, 33, 41, 6000])
def test_forest_deep_tree(rama, oracle32, n):
    # a long attractive path with a few repulsive chords: one tree as deep as the graph has nodes (the
    # small sizes put the deepest level on either side of the rooting loop's check interval)
    i = np.arange(n - 1, dtype=np.int32)
    j = i + 1
    rng = np.random.default_rng(3)
    c = rng.uniform(0.5, 1.5, n - 1).astype(np.float32)
    k = max(1, min(40, n // 8))
    span = max(3, min(200, n // 2))
    ci = rng.integers(0, n - span, k).astype(np.int32)
    cj = (ci + rng.integers(2, span, k)).astype(np.int32)
    ii, jj = np.concatenate([i, ci]), np.concatenate([j, cj])
    cc = np.concatenate([c, -np.ones(k, np.float32)])
    from paper_2109_01838_amd import default_params
    want = oracle32.contract(n, ii, jj, cc, repeat=1, forest_ratio=1.0)
    got = rama.contract(n, ii, jj, cc, params=default_params(forest_ratio=1.0), repeat=1)
    assert np.array_equal(np_(got["mapping"]), want["mapping"]) and got["n_nodes"] == want["n_nodes"]
    assert np.array_equal(np_(got["c"]), want["c"])


# runs of diagonal entries that end on either side of the 64 places a wave holds, and one much longer; ordered sums, so
# the result is the oracle's bit for bit
@pytest.mark.parametrize("sizes", [(1,), (2, 1, 2), (64,), (65,), (66, 2, 64), (33, 33), (32, 34, 3, 129, 2), (5000, 2, 700)])
def test_diagonal_of_long_runs(rama, oracle32, sizes):
    rng = np.random.default_rng(len(sizes))
    i, j, start = [], [], 0
    for k in sizes:                     # a path of k nodes, doubled by chords: contracted into one node
        i += list(range(start, start + k - 1)) + list(range(start, start + k - 2))
        j += list(range(start + 1, start + k)) + list(range(start + 2, start + k))
        start += k
    i, j = np.array(i, np.int32), np.array(j, np.int32)
    c = (rng.random(i.size) + 0.01).astype(np.float32)
    want = oracle32.contract(start, i, j, c, repeat=0)
    got = rama.contract(start, i, j, c, repeat=0)
    assert got["n_nodes"] == want["n_nodes"] == len(sizes)
    assert np.array_equal(np_(got["diag"]), want["diag"][: len(sizes)])


# the forest by one workgroup (and, from 32767 candidates on, by the whole chip); graphs beyond 6144 nodes, so that the
# round is not taken whole
@pytest.mark.parametrize("kind,n,m,cand", [("random", 20000, 40000, 1), ("random", 20000, 40000, 1024), ("random", 20000, 40000, 32767),
                                           ("random", 20000, 40000, 32768), ("random", 20000, 40000, 32769), ("path", 7000, 0, 0)])
def test_forest_in_one_workgroup(rama, oracle32, kind, n, m, cand):
    from paper_2109_01838_amd import default_params
    rng = np.random.default_rng(n + cand)
    if kind == "random":
        g = inputs.random_graph(n, m, 17)
        c = -np.abs(g["c"]) - np.float32(0.01)
        pick = rng.choice(c.size, cand, replace=False)
        c[pick] = np.round(-c[pick] * 4) / 4 + np.float32(0.25)      # a few values: ties decide
        i, j = g["i"], g["j"]
    else:                                                            # one tree as deep as the graph has nodes
        i = np.concatenate([np.arange(n - 1), np.arange(0, n - 50, 97)]).astype(np.int32)
        j = np.concatenate([np.arange(1, n), np.arange(0, n - 50, 97) + 41]).astype(np.int32)
        c = np.concatenate([rng.uniform(0.5, 1.5, n - 1), -np.ones(i.size - n + 1)]).astype(np.float32)
    want = oracle32.contract(n, i, j, c, repeat=1, forest_ratio=1.0)
    got = rama.contract(n, i, j, c, params=default_params(forest_ratio=1.0), repeat=1)
    assert got["n_nodes"] == want["n_nodes"] and np.array_equal(np_(got["mapping"]), want["mapping"])
    for k in ("i", "j", "c"):
        assert np.array_equal(np_(got[k]), want[k]), k


# the centres of the trees are their largest nodes: a sweep of the components joins one smaller node to each centre
@pytest.mark.parametrize("n,centres", [(3000, 1), (3000, 40), (7000, 1), (7000, 300)])
def test_components_of_trees_around_their_largest_nodes(rama, oracle32, n, centres):
    from paper_2109_01838_amd import default_params
    rng = np.random.default_rng(n + centres)
    leaves = np.arange(n - centres)
    i = np.concatenate([leaves, rng.choice(leaves, centres - 1, replace=False)])
    j = np.concatenate([n - centres + leaves % centres, n - centres + 1 + np.arange(centres - 1)])      # neighbouring trees share a leaf
    key = np.unique(i * n + j)
    i, j = (key // n).astype(np.int32), (key % n).astype(np.int32)
    c = (rng.integers(1, 5, key.size) / 4).astype(np.float32)
    want = oracle32.contract(n, i, j, c, repeat=1, forest_ratio=1.0)
    got = rama.contract(n, i, j, c, params=default_params(forest_ratio=1.0), repeat=1)
    assert got["n_nodes"] == want["n_nodes"] and np.array_equal(np_(got["mapping"]), want["mapping"])


# a list of more than 8192 candidates is not worked off by one workgroup, which takes up to 2.6 times as long
@pytest.mark.parametrize("cand", [8191, 8192, 8193])
def test_forest_in_one_workgroup_up_to_its_line(rama, oracle32, cand):
    from paper_2109_01838_amd import default_params
    test_forest_in_one_workgroup(rama, oracle32, "random", 20000, 40000, cand)
    g = inputs.random_graph(20000, 40000, 17)
    c = np.where(np.arange(g["c"].size) < cand, 1.0, -1.0).astype(np.float32)
    rama.profile_enable(True)
    rama.contract(g["n_nodes"], g["i"], g["j"], c, params=default_params(forest_ratio=1.0), repeat=1)
    names = {k["name"] for k in rama.profile_get()}
    rama.profile_enable(False)
    assert ("k_forest_short" in names) == (cand <= 8192), names


# --------------------------------------------------------------------------------------------
# whole rounds in one workgroup: graphs of up to 8192 edges and 6144 nodes
# --------------------------------------------------------------------------------------------
TAIL_SIZES = [(2, 1), (3, 3), (64, 63), (90, 1023), (90, 1024), (91, 1025), (700, 5000), (128, 8128), (3000, 8191), (3000, 8192),
              (3000, 8193), (6143, 8192), (6144, 8192), (6145, 8192)]


@pytest.mark.parametrize("n,m", TAIL_SIZES)
@pytest.mark.parametrize("repeat,ratio,pos", [(1, 0.1, 0.8), (0, 0.1, 0.6), (0, 1.0, 0.8), (0, 0.0, 0.9)])
def test_contraction_in_one_workgroup(rama, oracle32, n, m, repeat, ratio, pos):
    """Both sides of the limits; matching, forest and mixed; ties among the costs (a few values only)."""
    from paper_2109_01838_amd import default_params
    g = signed(inputs.random_graph(n, m, n + m), 5, pos)
    c = g["c"] if m % 2 else (np.round(g["c"] * 2) / 2).astype(np.float32)
    want = oracle32.contract(n, g["i"], g["j"], c, repeat=repeat, forest_ratio=ratio)
    got = rama.contract(n, g["i"], g["j"], c, params=default_params(forest_ratio=ratio), repeat=repeat)
    assert got["n_nodes"] == want["n_nodes"]
    assert np.array_equal(np_(got["mapping"]), want["mapping"])
    for k in ("i", "j", "c"):
        assert np.array_equal(np_(got[k]), want[k]), k
    assert np.array_equal(np_(got["diag"]), want["diag"][: got["n_nodes"]])


def test_graphs_without_attractive_edges_are_not_matched(rama, oracle32):
    """No candidates, and it is known: from the input's costs (parallel ones included), or from the separation of the last
    round.  Self-loops are no candidates either, and a threshold below zero may make some."""
    from paper_2109_01838_amd import default_params
    g = signed(inputs.random_graph(5000, 30000, 3, allow_messy=True), 4, 0.0)
    n, i, j, c = g["n_nodes"], g["i"], g["j"], g["c"]
    mixed = signed(inputs.random_graph(20000, 60000, 5), 6, 0.5)
    for kw, tau in ((dict(repeat=1), 0.0), (dict(repeat=0), 0.0), (dict(repeat=1), 0.5), (dict(repeat=1), -0.3)):
        want = oracle32.contract(n, i, j, c, tau=tau, **kw)
        rama.profile_enable(True)
        got = rama.contract(n, i, j, c, params=default_params(contract_threshold=tau), **kw)
        names = {k["name"] for k in rama.profile_get()}
        rama.profile_enable(False)
        assert ("k_handshake_finish" in names) == (tau < 0.0)
        assert got["n_nodes"] == want["n_nodes"] and np.array_equal(np_(got["mapping"]), want["mapping"])
        for k in ("i", "j", "c"):
            assert np.array_equal(np_(got[k]), want[k]), k
    # a whole solve: its last round on more edges than one workgroup takes
    rama.profile_enable(True)
    got = rama.solve(mixed["n_nodes"], mixed["i"], mixed["j"], mixed["c"])
    launches = sum(k["launches"] for k in rama.profile_get() if k["name"] == "k_handshake_finish")
    rama.profile_enable(False)
    want = oracle32.solve(mixed["n_nodes"], mixed["i"], mixed["j"], mixed["c"])
    assert np.array_equal(np_(got["labels"]), want["labels"]) and got["rounds"] == want["rounds"]
    last = rama.round_stats()[-1]
    assert last["n_attractive"] == 0 and last["n_contracted"] == 0 and last["n_edges"] > 8192
    assert launches == sum(r["n_contracted"] > 0 for r in rama.round_stats())


# rows of the candidate list that fill a wave, span two, or are broken up by edges that are no candidates; the costs leave the
# best candidate of a row at its front, at its end and in the middle
@pytest.mark.parametrize("degree", [1, 2, 3, 4, 33, 63, 64, 65, 127, 128, 300])
@pytest.mark.parametrize("pos", [1.0, 0.6])
@pytest.mark.parametrize("slope", [-1, 0, 1])
def test_rows_of_the_first_proposals(rama, oracle32, degree, pos, slope):
    rows = 9000 // degree + 3
    rng = np.random.default_rng(degree)
    i = np.repeat(np.arange(rows), degree)
    j = rows + rng.integers(0, 4 * rows, i.size)
    c = 1.0 + slope * np.tile(np.arange(degree), rows) / (2.0 * degree) + (0.0 if slope else 1.0) * rng.random(i.size)
    c = (c * np.where(rng.random(i.size) < pos, 1, -1)).astype(np.float32)
    n = 5 * rows
    want = oracle32.contract(n, i.astype(np.int32), j.astype(np.int32), c, repeat=1)
    got = rama.contract(n, i.astype(np.int32), j.astype(np.int32), c, repeat=1)
    assert got["n_nodes"] == want["n_nodes"] and np.array_equal(np_(got["mapping"]), want["mapping"])
    for k in ("i", "j", "c"):
        assert np.array_equal(np_(got[k]), want[k]), k


# The last workgroup of a matching: rank words by node (up to 16384) and by hash (twice as many places to find for lists of up
# to 4096), full lists of edges without a common node, paths of ascending costs (a pair a handshake, more of them than the cap
# allows), nodes that fill their last row of 64 or begin one, both sides of the 32768 it numbers
@pytest.mark.parametrize("n,m,kind", [(2, 1, "path"), (65, 40, "path"), (1023, 1022, "path"), (1024, 1023, "path"), (1025, 1024, "path"),
                                      (16384, 8192, "pairs"), (16384, 8192, "path"), (16385, 4096, "pairs"), (16385, 4096, "path"),
                                      (16385, 4097, "path"), (32768, 4096, "pairs"), (32768, 4095, "random"), (32769, 4096, "random"),
                                      (16384, 9000, "random"), (16385, 9000, "random"), (300, 8192, "random"), (200000, 4096, "spread"),
                                      # more rounds than there are counters for at a time, of lists that stay long
                                      (20001, 20000, "path"), (1100001, 1100000, "path")])
@pytest.mark.parametrize("cap", [32, 3])
def test_last_workgroup_of_a_matching(rama, oracle32, n, m, kind, cap):
    from paper_2109_01838_amd import default_params
    rng = np.random.default_rng(n + m)
    if kind == "path":
        i, j, c = np.arange(m), np.arange(1, m + 1), np.linspace(1, 2, m)
    elif kind == "pairs":
        i, j, c = 2 * np.arange(m), 2 * np.arange(m) + 1, 1 + rng.random(m)
    else:
        i, j = rng.integers(0, n, m), rng.integers(0, n, m)
        c = np.round(8 * rng.random(m) + 1) / 8 if kind == "random" else 1 + rng.random(m)
        if kind == "spread":      # a node of few in many: the table's places are far apart
            i = i // 97 * 97
    i, j, c = i.astype(np.int32), j.astype(np.int32), c.astype(np.float32)
    want = oracle32.contract(n, i, j, c, repeat=1, rounds_cap=cap, forest_ratio=0.0)
    got = rama.contract(n, i, j, c, params=default_params(matching_rounds_cap=cap, forest_ratio=0.0), repeat=1)
    assert got["n_nodes"] == want["n_nodes"] and np.array_equal(np_(got["mapping"]), want["mapping"])
    for k in ("i", "j", "c"):
        assert np.array_equal(np_(got[k]), want[k]), k


# Contraction with a workgroup to a digit: lists on both sides of the tiles (1024 edges up to 196608, 2048 beyond); parallel
# edges that fill buckets of the in-LDS sort, rows far apart and close together (the bits of hi - lo), digits without an edge,
# and lists that are too long for it, on both sides of 2^21 edges (its own lines: test_lines_of_contraction_by_digits)
@pytest.mark.parametrize("n,m,near", [(3000, 8193, 0), (3000, 9217, 5), (200, 19000, 0), (150, 8300, 0), (70000, 196608, 4), (70000, 196609, 4),
                                      (5000, 197633, 0), (1000000, 300000, 2), (1048577, 300000, 0), (600, 170000, 0), (40000, 2097151, 0), (40000, 2097153, 0)])
@pytest.mark.parametrize("ratio", [0.0, 1.0], ids=["matching", "forest"])
def test_contraction_by_digits(rama, oracle32, n, m, near, ratio):
    from paper_2109_01838_amd import default_params
    if ratio and m > 400000:
        pytest.skip("the oracle's forest takes its time")
    rng = np.random.default_rng(n + m)
    i = rng.integers(0, n, 2 * m)
    j = (i + rng.integers(1, near + 1, i.size)) % n if near else rng.integers(0, n, i.size)
    key = np.unique(np.minimum(i, j) * np.int64(n) + np.maximum(i, j))
    key = key[key // n != key % n]
    key = np.sort(rng.permutation(key)[:m])
    i, j = (key // n).astype(np.int32), (key % n).astype(np.int32)
    c = (np.round(rng.random(i.size) * 16 - 6) / 8).astype(np.float32)
    want = oracle32.contract(n, i, j, c, repeat=1, forest_ratio=ratio)
    got = rama.contract(n, i, j, c, params=default_params(forest_ratio=ratio), repeat=1)
    assert got["n_nodes"] == want["n_nodes"] and np.array_equal(np_(got["mapping"]), want["mapping"])
    for k in ("i", "j", "c"):
        assert np.array_equal(np_(got[k]), want[k]), k
    assert np.array_equal(np_(got["diag"]), want["diag"][: got["n_nodes"]])


def pairs_and_more(n_new, m, pairs, seed):
    """m edges of n_new + pairs nodes, between nodes that are close, of which only those of `pairs` pairs of neighbours attract:
    what a matching and a forest contract.  Half of the others come in twos that are parallel behind it."""
    rng = np.random.default_rng(seed)
    n = n_new + pairs
    first = np.arange(pairs, dtype=np.int64) * (n - 1) // pairs
    p, x = rng.choice(first, m), rng.integers(0, n, 2 * m)
    twos, near = p + rng.integers(2, 800, m), x + rng.integers(1, 800, x.size)
    key = np.stack([p * n + twos, (p + 1) * n + twos], axis=1)[twos < n][: m // 4].ravel()
    inner = first * n + first + 1
    key = np.concatenate([key, (x * n + near)[near < n]])
    key = key[np.sort(np.unique(key, return_index=True)[1])]       # the twos first
    key = key[~np.isin(key, inner)][:m - pairs]
    assert key.size == m - pairs
    c = np.concatenate([1 + rng.random(pairs), -(rng.integers(1, 9, key.size) / 8)])
    key = np.concatenate([inner, key])
    order = np.argsort(key)
    key, c = key[order], c[order]
    return n, (key // n).astype(np.int32), (key % n).astype(np.int32), c.astype(np.float32)


# Both sides of the lines of contraction by digits, which comes for lists of more than 8192 edges if the bits of a new node's
# number and those of a row that are left behind at most eight bits of a digit fit 32, and a digit has at most 4096 edges on average:
# 2^20 edges where the nodes use 256 digits up, 528384 where they are just enough for one bit more and use 129
@pytest.mark.parametrize("n_new,m,digits", [(6900, 8192, False), (6900, 8193, True), (65536, 1 << 20, True), (65536, (1 << 20) + 1, False),
                                            (32769, 528384, True), (32769, 528385, False), (1 << 20, 300000, True), ((1 << 20) + 1, 300000, False)])
@pytest.mark.parametrize("ratio", [0.0, 1.0], ids=["matching", "forest"])
def test_lines_of_contraction_by_digits(rama, oracle32, n_new, m, digits, ratio):
    from paper_2109_01838_amd import default_params
    n, i, j, c = pairs_and_more(n_new, m, 2000, m)
    want = oracle32.contract(n, i, j, c, repeat=1, forest_ratio=ratio)
    rama.profile_enable(True)
    got = rama.contract(n, i, j, c, params=default_params(forest_ratio=ratio), repeat=1)
    names = {k["name"] for k in rama.profile_get()}
    rama.profile_enable(False)
    assert ("k_join_digits" in names) == digits and ("k_relabel_keys" in names) == (not digits)
    assert got["n_nodes"] == want["n_nodes"] == n_new and np.array_equal(np_(got["mapping"]), want["mapping"])
    assert want["i"].size < m - 2000
    for k in ("i", "j", "c"):
        assert np.array_equal(np_(got[k]), want[k]), k
    assert np.array_equal(np_(got["diag"]), want["diag"][:n_new])


@pytest.mark.parametrize("leaves,fits", [(8000, True), (8192, True), (8193, False), (12000, False)])
def test_matching_that_crowds_a_digit(rama, oracle32, leaves, fits):
    """One row with all that a workgroup sorts in LDS, or more, behind a matching: the contraction by digits gives up, the edges
    are relabelled once more, and the diagonal is written twice."""
    from paper_2109_01838_amd import default_params
    n, i, j, c = pairs_and_more(60000, 70000, 2000, leaves)
    keep = (i >= 1100) | (c > 0)                           # the digit of the first 1024 new nodes is the hub's alone
    hub, leaf = 0, 4000 + np.arange(leaves)                # it is contracted with 1
    i, j = np.concatenate([i[keep], np.full(leaves, hub)]), np.concatenate([j[keep], leaf])
    c = np.concatenate([c[keep], -1 - np.arange(leaves) / leaves])
    order = np.lexsort((j, i))
    i, j, c = i[order].astype(np.int32), j[order].astype(np.int32), c[order].astype(np.float32)
    want = oracle32.contract(n, i, j, c, repeat=1, forest_ratio=0.0)
    assert 0 <= leaves - np.bincount(want["i"])[:1024].sum() < leaves // 10
    rama.profile_enable(True)
    got = rama.contract(n, i, j, c, params=default_params(forest_ratio=0.0), repeat=1)
    names = {k["name"] for k in rama.profile_get()}
    rama.profile_enable(False)
    assert "k_join_digits" in names and ("k_relabel_keys" in names) == (not fits)
    assert got["n_nodes"] == want["n_nodes"] == 60000 and np.array_equal(np_(got["mapping"]), want["mapping"])
    for k in ("i", "j", "c"):
        assert np.array_equal(np_(got[k]), want[k]), k
    assert np.array_equal(np_(got["diag"]), want["diag"][:60000]) and np.count_nonzero(want["diag"]) == 2000


def test_contraction_leaves_nothing(rama, oracle32):
    """A clique whose edges all attract, as a forest: one node is left, and no edge."""
    from paper_2109_01838_amd import default_params
    n = 200
    i, j = np.triu_indices(n, 1)
    c = np.linspace(1, 2, i.size).astype(np.float32)
    got = rama.contract(n, i.astype(np.int32), j.astype(np.int32), c, params=default_params(forest_ratio=1.0), repeat=1)
    assert got["n_nodes"] == 1 and got["i"].numel() == 0 and not np_(got["mapping"]).any()


# Both sides of the lines up to which the matching's last workgroup numbers the nodes (2^15 nodes) and nobody
# waits for the number of candidates or of kept edges (2^20 edges, all different: parallel ones are added up before); every
# edge a candidate, none, and too many candidates left for the last workgroup behind the rounds that should bring them there (a star keeps all of them)
@pytest.mark.parametrize("n,m,pos", [(32768, 60000, 0.8), (32769, 60000, 0.8), (8193, 40000, 0.5), (20000, 1 << 20, 0.6), (20000, (1 << 20) + 1, 0.6),
                                     (9000, 30000, 1.0), (9000, 30000, 0.0), (70000, 60000, -1.0), (2, 9000, 1.0)])
def test_contraction_that_waits_for_no_counts(rama, oracle32, n, m, pos):
    rng = np.random.default_rng(n + m)
    if pos < 0:      # a star, its costs ascending: a handshake round matches one pair, the others propose again
        i, j = np.zeros(n - 1, np.int32), np.arange(1, n, dtype=np.int32)
        i, j = np.concatenate([i, rng.integers(1, n, m)]).astype(np.int32), np.concatenate([j, rng.integers(1, n, m)]).astype(np.int32)
        c = np.concatenate([np.linspace(1, 2, n - 1), np.linspace(0.1, 0.9, m)]).astype(np.float32)
    else:
        i, j = rng.integers(0, n, m).astype(np.int32), rng.integers(0, n, m).astype(np.int32)
        if m >= 1 << 20:
            g = inputs.random_graph(n, m, n + m)
            i, j = g["i"], g["j"]
            assert i.size == m and np.unique(i * np.int64(n) + j).size == m
        c = (np.round(rng.random(m) * 8 + 1) / 8 * np.where(rng.random(m) < pos, 1, -1)).astype(np.float32)
    want = oracle32.contract(n, i, j, c, repeat=1)
    got = rama.contract(n, i, j, c, repeat=1)
    assert got["n_nodes"] == want["n_nodes"] and np.array_equal(np_(got["mapping"]), want["mapping"])
    for k in ("i", "j", "c"):
        assert np.array_equal(np_(got[k]), want[k]), k


@pytest.mark.parametrize("leaves", [8192, 8193, 20000])
def test_contraction_that_crowds_a_row(rama, oracle32, leaves):
    """The input's edges are in order and need no sort; a forest joins 2000 nodes into one, whose row is then as long as what a
    workgroup sorts in LDS, or longer: nobody knew how many edges would be kept, and they are sorted once more."""
    from paper_2109_01838_amd import default_params
    rng = np.random.default_rng(leaves)
    hub, n = 2000, 2000 + leaves + 9000
    leaf = hub + np.arange(leaves)
    rest = np.unique(np.sort(rng.integers(hub + 1024, n, (60000, 2)), axis=1), axis=0)      # their rows have digits of their own
    rest = rest[rest[:, 0] < rest[:, 1]]
    i = np.concatenate([np.arange(hub - 1), leaf % hub, rest[:, 0]])
    j = np.concatenate([np.arange(1, hub), leaf, rest[:, 1]])
    c = np.concatenate([100.0 + rng.random(hub - 1), -rng.random(leaves + rest.shape[0]) - 0.01])
    order = np.lexsort((j, i))
    i, j, c = i[order].astype(np.int32), j[order].astype(np.int32), c[order].astype(np.float32)
    rama.profile_enable(True)
    got = rama.contract(n, i, j, c, params=default_params(forest_ratio=1.0), repeat=1)
    passes = sum(x["launches"] for x in rama.profile_get() if x["name"].startswith("k_rs_hist"))
    rama.profile_enable(False)
    want = oracle32.contract(n, i, j, c, repeat=1, forest_ratio=1.0)
    assert got["n_nodes"] == want["n_nodes"] == n - hub + 1 and np.array_equal(np_(got["mapping"]), want["mapping"])
    for k in ("i", "j", "c"):
        assert np.array_equal(np_(got[k]), want[k]), k
    row, others = int((np_(got["i"]) == 0).sum()), int((np_(got["i"]) != 0).sum())
    assert row == leaves and others > 50000
    assert passes == 1 if leaves <= 8192 else passes > 2


@pytest.mark.parametrize("n,m,pos", [(64, 300, 0.7), (90, 2000, 0.9), (128, 8128, 0.75), (128, 8128, 0.97), (1000, 8000, 0.8), (4000, 8200, 0.9),
                                     (400, 6000, 0.9), (8000, 20000, 0.85)])
@pytest.mark.parametrize("later,iters,max_rounds", [(3, 5, 0), (3, 1, 3), (0, 0, 0), (3, 12, 2)])
def test_solve_rounds_in_one_workgroup(rama, oracle32, n, m, pos, later, iters, max_rounds):
    """Rounds behind the first on small graphs, with and without triangles (up to and beyond the 2048 that fit)."""
    from paper_2109_01838_amd import default_params
    g = signed(inputs.random_graph(n, m, 3 * n + m), 9, pos)
    want = oracle32.solve(n, g["i"], g["j"], g["c"], max_cycle_len_first=3, max_cycle_len_later=later, mp_iters_first=2, mp_iters_later=iters,
                          max_rounds=max_rounds)
    p = default_params(max_cycle_len_first=3, max_cycle_len_later=later, mp_iters_first=2, mp_iters_later=iters, max_rounds=max_rounds)
    got = rama.solve(n, g["i"], g["j"], g["c"], p)
    assert got["rounds"] == want["rounds"] and got["n_clusters"] == want["n_clusters"]
    assert np.array_equal(np_(got["labels"]), want["labels"])
    assert rel_close(got["primal"], want["primal"], 1e-9) and rel_close(got["lower_bound"], want["lower_bound"], 1e-6)
    rounds = rama.round_stats()
    assert len(rounds) == got["rounds"] and rounds[-1]["n_edges_aug"] >= got["n_edges_final"]


# one-workgroup rounds without triangles that contract a book of `pages` pages and a star of up to `leaves` leaves
@pytest.mark.parametrize("pages,leaves", [(47, 10), (48, 159), (49, 161), (50, 400), (200, 1000), (600, 5000), (3, 6000)])
def test_long_rows_and_runs_in_one_workgroup(rama, oracle32, pages, leaves):
    from paper_2109_01838_amd import default_params
    rng = np.random.default_rng(pages + leaves)
    page = 2 + np.arange(pages)
    hub = 2 + pages
    leaf = hub + 1 + np.arange(min(leaves, 6140 - hub))
    spare = leaf[-1] + 1
    i = np.concatenate([[0], np.zeros(pages), np.ones(pages), np.full(leaf.size, hub), [spare]]).astype(np.int32)
    j = np.concatenate([[1], page, page, leaf, [spare + 1]]).astype(np.int32)
    c = np.concatenate([[-50.0], 1 + rng.random(2 * pages), rng.random(leaf.size) - 0.5, [5.0]]).astype(np.float32)
    for later in (3, 0):
        kw = dict(max_cycle_len_first=0, mp_iters_first=0, max_cycle_len_later=later, mp_iters_later=4, max_rounds=6)
        want = oracle32.solve(int(spare + 2), i, j, c, **kw)
        got = rama.solve(int(spare + 2), i, j, c, params=default_params(**kw))
        assert np.array_equal(np_(got["labels"]), want["labels"]) and got["rounds"] == want["rounds"]


# One-workgroup rounds whose messages go by comparing (an edge of up to 48 slots) and by sorts (more): a repulsive edge in `pages`
# triangles, whose other edges are in one to three.  The first round contracts every node with one of its own, so that the second
# one, the first in one workgroup, has the book as it is.  What is contracted then, and when, depends on the messages.
@pytest.mark.parametrize("pages", [3, 47, 48, 49, 50, 200, 680])
def test_messages_of_long_runs_in_one_workgroup(rama, oracle32, pages):
    from paper_2109_01838_amd import default_params
    rng = np.random.default_rng(pages)
    page, nodes = 2 + np.arange(pages), np.arange(2 + pages)
    i = np.concatenate([[0], np.zeros(pages), np.ones(pages), page[:-1], nodes]).astype(np.int32)
    j = np.concatenate([[1], page, page, page[1:], nodes.size + nodes]).astype(np.int32)
    c = np.concatenate([[-0.4 * pages], 1 + rng.random(2 * pages), -0.2 - rng.random(pages - 1), 100 + rng.random(nodes.size)]).astype(np.float32)
    n = 2 * nodes.size
    second = oracle32.contract(n, i, j, c, repeat=1, rounds_cap=1, forest_ratio=0.0)
    tri = oracle32.find_conflicted_cycles(second["n_nodes"], second["i"], second["j"], second["c"], 3)[0]
    sides = np.sort(np.concatenate([tri[:, :2], tri[:, 1:], tri[:, ::2]]), axis=1)
    slots = np.unique(sides[:, 0] * nodes.size + sides[:, 1], return_counts=True)[1]
    assert slots.max() == pages and tri.shape[0] == 3 * pages - 2 <= 2048
    kw = dict(max_cycle_len_first=0, mp_iters_first=0, max_cycle_len_later=3, matching_rounds_cap=1, forest_ratio=0.0)
    want, without = (oracle32.solve(n, i, j, c, mp_iters_later=k, **kw) for k in (4, 0))
    assert pages == 3 or not np.array_equal(want["labels"], without["labels"])
    rama.profile_enable(True)
    got = rama.solve(n, i, j, c, params=default_params(mp_iters_later=4, **kw))
    names = {k["name"] for k in rama.profile_get()}
    rama.profile_enable(False)
    rounds = rama.round_stats()
    assert "k_tail_rounds" in names and rounds[1]["n_edges"] == second["i"].size and rounds[1]["n_triangles"] == tri.shape[0]
    assert np.array_equal(np_(got["labels"]), want["labels"]) and got["rounds"] == want["rounds"]
    assert got["n_edges_final"] == want["n_edges_final"] and rel_close(got["primal"], want["primal"], 1e-9)


# Contraction in one workgroup on both sides of the 160 keys that a bucket of its sort may hold: with 2049 to 4096 nodes left a
# bucket is a row, and the longest row is the hub's, `twice` of whose edges are parallel to another one
@pytest.mark.parametrize("row,twice", [(159, 0), (160, 0), (160, 60), (161, 0), (161, 61), (2500, 300)])
@pytest.mark.parametrize("n_new", [2049, 4096])
def test_rows_that_fill_a_bucket_in_one_workgroup(rama, oracle32, row, twice, n_new):
    from paper_2109_01838_amd import default_params
    rng = np.random.default_rng(row + n_new)
    row = min(row, n_new - 400)
    pairs = 400 + twice                    # nodes 2k + 1 and 2k + 2, k < pairs
    n = n_new + pairs
    assert n <= 6144
    leaf = np.concatenate([1 + 2 * np.arange(twice), 2 + 2 * np.arange(twice), 2 * pairs + 1 + rng.permutation(n - 2 * pairs - 1)[:row - 2 * twice]])
    inner, far = 1 + 2 * np.arange(pairs), rng.integers(1, n, (2000, 2))
    i, j = np.concatenate([inner, np.zeros(leaf.size, np.int64), far[:, 0]]), np.concatenate([inner + 1, leaf, far[:, 1]])
    i, j = np.minimum(i, j), np.maximum(i, j)
    c = np.concatenate([1 + rng.random(pairs), -0.1 - rng.random(i.size - pairs)]).astype(np.float32)
    first = np.unique(i.astype(np.int64) * n + j, return_index=True)[1]
    first = first[i[first] != j[first]]
    i, j, c = i[first].astype(np.int32), j[first].astype(np.int32), c[first]
    want = oracle32.contract(n, i, j, c, repeat=1, forest_ratio=0.0)
    assert want["n_nodes"] == n_new and i.size <= 8192
    a, b = want["mapping"][i], want["mapping"][j]
    rows = np.bincount(np.minimum(a, b)[a != b])
    assert rows[0] == rows.max() == row and want["i"].size <= np.count_nonzero(a != b) - twice
    got = rama.contract(n, i, j, c, params=default_params(forest_ratio=0.0), repeat=1)
    assert np.array_equal(np_(got["mapping"]), want["mapping"])
    for k in ("i", "j", "c"):
        assert np.array_equal(np_(got[k]), want[k]), k


@pytest.mark.parametrize("n,m,pos", [(200, 8100, 0.7), (700, 8100, 0.8)])
def test_dense_rounds_are_handed_back(rama, oracle32, n, m, pos):
    """Rounds of more than 2048 triangles are not for one workgroup: it gets another try only behind a round of 16384 or
    fewer."""
    from paper_2109_01838_amd import default_params
    rng = np.random.default_rng(1)
    i, j = np.triu_indices(n, 1)
    k = np.sort(rng.permutation(i.size)[:m])
    i, j = i[k].astype(np.int32), j[k].astype(np.int32)
    c = ((rng.random(m) + 0.01) * np.where(rng.random(m) < pos, 1, -1)).astype(np.float32)
    want = oracle32.solve(n, i, j, c, max_cycle_len_first=3)
    rama.profile_enable(True)
    got = rama.solve(n, i, j, c, params=default_params(max_cycle_len_first=3))
    launches = sum(x["launches"] for x in rama.profile_get() if x["name"] == "k_tail_rounds")
    rama.profile_enable(False)
    assert np.array_equal(np_(got["labels"]), want["labels"])
    rounds, tries, try_next = [r["n_triangles"] for r in rama.round_stats()[1:]], 0, True
    assert any(a > 16384 and b > 2048 for a, b in zip(rounds, rounds[1:]))
    while rounds:
        if try_next:
            tries += 1
            while rounds and rounds[0] <= 2048:
                rounds.pop(0)
        if rounds:
            try_next = rounds.pop(0) <= 16384
    assert launches == tries


def test_contract_fig2_graph(rama, oracle32):
    # the graph of the paper's Fig. 2; with the matching rule S={st} (cost 4 is the best edge at s and t;
    # rs=3 loses at s), so only the mechanics are compared with the oracle here
    i = np.array([0, 0, 1, 1, 2, 3, 2], np.int32)
    j = np.array([1, 2, 3, 4, 3, 4, 4], np.int32)
    c = np.array([1, -2, -3, 1, 3, 4, 1], np.float32)
    want = oracle32.contract(5, i, j, c, repeat=1)
    got = rama.contract(5, i, j, c, repeat=1)
    assert np.array_equal(np_(got["mapping"]), want["mapping"])
    assert np.array_equal(np_(got["c"]), want["c"]) and np.array_equal(np_(got["diag"]), want["diag"])


def test_canonicalisation_of_large_shuffled_input(rama, oracle32):
    # no attractive edge -> rama_contract returns the canonical form of its input: this drives the
    # 64-bit radix sort, the run reduction and the scans over many tiles with a ragged tail
    g = inputs.random_graph(3000, 100003, 21, allow_messy=True)
    c = -np.abs(g["c"]) - 0.01
    wi, wj, wc = oracle32.canonicalise(3000, g["i"], g["j"], c)
    got = rama.contract(3000, g["i"], g["j"], c, repeat=1)
    assert got["n_nodes"] == 3000 and np.array_equal(np_(got["mapping"]), np.arange(3000))
    assert np.array_equal(np_(got["i"]), wi) and np.array_equal(np_(got["j"]), wj)
    assert np.array_equal(np_(got["c"]), wc)       # duplicates are added in input order on both sides


# Arrays that one workgroup sorts in LDS, ordered by one comparison of a key's low bits and its place while those fit a word
# (32 bits of key do not, 31 do), and by passes where a bucket of equal top bits is long (few nodes)
@pytest.mark.parametrize("n,m,bits", [(1 << 16, 8192, 32), (50000, 8191, 32), (50000, 8192, 31), (32768, 8192, 30), (20000, 8192, 30), (300, 4097, 18),
                                      (70, 8192, 14), (3, 8192, 4), (1 << 20, 4096, 40)])
def test_sort_inside_one_workgroup(rama, oracle32, n, m, bits):
    rng = np.random.default_rng(n + m)
    i = rng.integers(0, n, m).astype(np.int32)
    j = ((i + 1 + rng.integers(0, n - 1, m)) % n).astype(np.int32)
    far = min(n - 1, (1 << bits - (n - 1).bit_length()) - 1)            # the widest second field
    j = np.clip(j, i - far, i + far).astype(np.int32)
    i[0], j[0] = 0, far
    assert (n - 1).bit_length() + int(np.abs(i.astype(np.int64) - j).max()).bit_length() == bits
    c = (-np.abs(rng.normal(size=m)) * 10.0 ** rng.integers(-3, 4, m) - 1e-3).astype(np.float32)
    wi, wj, wc = oracle32.canonicalise(n, i, j, c)
    got = rama.contract(n, i, j, c, repeat=1, want_diag=False)
    assert np.array_equal(np_(got["i"]), wi) and np.array_equal(np_(got["j"]), wj) and np.array_equal(np_(got["c"]), wc)


# lengths at which the radix passes change their tiles (1024 or 2048 keys, 6144 / 5120 beyond), and one key more or less
# than whole tiles of each
@pytest.mark.parametrize("m", [8193, 33 * 1024, 196608, 196609, 200 * 2048 + 1, 3145728, 3145729, 513 * 6144 + 1])
def test_sort_at_the_limits_of_its_tiles(rama, oracle32, m):
    rng = np.random.default_rng(m)
    n = 1 << 20
    i, j = rng.integers(0, n, m).astype(np.int32), rng.integers(0, n, m).astype(np.int32)
    c = -rng.random(m, dtype=np.float32) - np.float32(0.01)
    wi, wj, wc = oracle32.canonicalise(n, i, j, c)
    got = rama.contract(n, i, j, c, repeat=1, want_diag=False)      # no attractive edge: the canonical form of the input
    assert np.array_equal(np_(got["i"]), wi) and np.array_equal(np_(got["j"]), wj) and np.array_equal(np_(got["c"]), wc)


# One pass over the top bits and one in-LDS sort, a workgroup to a digit: `crowd` keys with the same digit, as many as a
# workgroup holds (8192; 4096 of 64 bits) and one more, in front, in the middle and at the end of the others
@pytest.mark.parametrize("n,m,crowd,at", [(40000, 30000, 8192, 0.5), (40000, 30000, 8193, 0.5), (40000, 30000, 8193, 0.0), (40000, 30000, 9000, 1.0),
                                          (1 << 21, 12000, 4096, 0.5), (1 << 21, 12000, 4097, 0.5), (40000, 393216, 0, 0.0), (40000, 900000, 20000, 0.3)])
def test_sort_that_may_find_out_later(rama, oracle32, n, m, crowd, at):
    rng = np.random.default_rng(n + m + crowd)
    i, j = rng.integers(0, n, m).astype(np.int32), rng.integers(0, n, m).astype(np.int32)
    lone = max(0, min(n - 2, int(at * n) - 1))
    i[i == lone] = (lone + 1) % n                                       # nobody else's row
    here = rng.permutation(m)[:crowd]
    i[here], j[here] = lone, rng.integers(lone + 1, n, crowd)
    i[0], j[0] = 0, n - 1
    c = (-np.abs(rng.normal(size=m)) * 10.0 ** rng.integers(-3, 4, m) - 1e-3).astype(np.float32)
    wi, wj, wc = oracle32.canonicalise(n, i, j, c)
    got = rama.contract(n, i, j, c, repeat=1, want_diag=False)
    assert np.array_equal(np_(got["i"]), wi) and np.array_equal(np_(got["j"]), wj) and np.array_equal(np_(got["c"]), wc)


@pytest.mark.parametrize("n,m", [(3, 20001), (2, 2049), (5, 4096), (40, 70000)])
def test_canonicalisation_sums_long_runs_in_input_order(rama, oracle32, n, m):
    # few nodes, many parallel edges: every run of equal pairs is thousands of entries long and crosses
    # the 2048-entry tiles of the run reduction, some exactly at a tile's end; costs of mixed magnitude
    # make the float sum depend on the order of the adds
    rng = np.random.default_rng(n * 1000 + m)
    i = rng.integers(0, n, m).astype(np.int32)
    j = ((i + 1 + rng.integers(0, max(n - 1, 1), m)) % n).astype(np.int32)
    c = (-np.abs(rng.normal(size=m)) * 10.0 ** rng.integers(-3, 4, m) - 1e-3).astype(np.float32)
    wi, wj, wc = oracle32.canonicalise(n, i, j, c)
    got = rama.contract(n, i, j, c, repeat=1)
    assert np.array_equal(np_(got["i"]), wi) and np.array_equal(np_(got["j"]), wj)
    assert np.array_equal(np_(got["c"]), wc)


@pytest.mark.parametrize("runs", [2, 3, 5, 8, 9])
def test_canonicalisation_of_a_few_sorted_runs(rama, oracle32, runs):
    # an edge list made of `runs` sorted pieces (as a grid written direction by direction): up to eight pieces are
    # merged instead of sorted; pairs that occur in several pieces, flipped pairs and self-loops included
    rng = np.random.default_rng(100 + runs)
    n, m = 40000, 120000
    a = rng.integers(0, n, m); b = rng.integers(0, n, m)
    loops = rng.random(m) < 0.01
    b = np.where(loops, a, b)
    lo, hi = np.minimum(a, b), np.maximum(a, b)
    piece = rng.integers(0, runs, m)
    dup = rng.random(m) < 0.1                                    # a tenth of the pairs also goes into another piece
    lo = np.concatenate([lo, lo[dup]]); hi = np.concatenate([hi, hi[dup]])
    piece = np.concatenate([piece, (piece[dup] + 1) % runs])
    order = np.lexsort((hi, lo, piece))                          # piece by piece, each sorted by (lo, hi)
    lo, hi = lo[order], hi[order]
    flip = rng.random(lo.size) < 0.3
    i = np.where(flip, hi, lo).astype(np.int32); j = np.where(flip, lo, hi).astype(np.int32)
    c = (-np.abs(rng.normal(size=i.size)) * 10.0 ** rng.integers(-2, 3, i.size) - 1e-3).astype(np.float32)
    wi, wj, wc = oracle32.canonicalise(n, i, j, c)
    got = rama.contract(n, i, j, c, repeat=1)                    # no attractive edge: the canonical form comes back
    assert np.array_equal(np_(got["i"]), wi) and np.array_equal(np_(got["j"]), wj)
    assert np.array_equal(np_(got["c"]), wc)


# sorted pieces without repeated pairs are interleaved in one pass over ranges of nodes; a pair in two pieces, a node with
# more than 64 edges, more edges than a range holds (3072) and more than 16 pieces take the general way
@pytest.mark.parametrize("runs,kind", [(1, "plain"), (2, "plain"), (3, "plain"), (15, "plain"), (16, "plain"), (17, "plain"), (3, "dup"),
                                       (3, "row64"), (3, "row65"), (4, "crowded"), (3, "sparse"), (3, "tiny")])
def test_canonicalisation_interleaves_sorted_runs(rama, oracle32, runs, kind):
    rng = np.random.default_rng(200 + runs)
    n, m = {"sparse": (400000, 9000), "tiny": (900, 4097)}.get(kind, (20011, 90000))
    a, b = rng.integers(0, n, 2 * m), rng.integers(0, n, 2 * m)
    if kind == "crowded":                                        # most edges at a few nodes, none of them with many
        a[: m] = rng.integers(5000, 5200, m)
    lo, hi = np.minimum(a, b), np.maximum(a, b)
    if kind.startswith("row"):
        k = int(kind[3:])
        keep = lo != 7
        lo, hi = np.concatenate([lo[keep], np.full(k, 7)]), np.concatenate([hi[keep], 100 + 3 * np.arange(k)])
    key = np.unique(lo[lo != hi].astype(np.int64) * n + hi[lo != hi])
    if kind == "crowded":
        cnt = np.concatenate([np.arange(x) for x in np.bincount((key // n).astype(np.int64), minlength=n)])
        key = key[cnt < 60]
    if not kind.startswith("row"):
        key = np.sort(rng.permutation(key)[:m])
    piece = rng.integers(0, runs, key.size)
    if kind == "dup":
        key, piece = np.append(key, key[1234]), np.append(piece, (piece[1234] + 1) % runs)
    order = np.lexsort((key, piece))
    lo, hi = key[order] // n, key[order] % n
    flip = rng.random(lo.size) < 0.3
    i, j = np.where(flip, hi, lo).astype(np.int32), np.where(flip, lo, hi).astype(np.int32)
    c = (-np.abs(rng.normal(size=i.size)) - 1e-3).astype(np.float32)
    c[rng.random(i.size) < 0.1] = 0.0
    wi, wj, wc = oracle32.canonicalise(n, i, j, c)
    got = rama.contract(n, i, j, c, repeat=1, want_diag=False)
    assert np.array_equal(np_(got["i"]), wi) and np.array_equal(np_(got["j"]), wj) and np.array_equal(np_(got["c"]), wc)
    # the signs the pass counts on its way are the ones the separation splits the edges by
    c = np.where(rng.random(i.size) < 0.6, 1.0, -1.0).astype(np.float32)
    want = oracle32.find_conflicted_cycles(n, i, j, c, 3)
    assert np.array_equal(np_(rama.find_conflicted_cycles(n, i, j, c, 3)[0]), want[0])


# the first pass of the sort takes the edges themselves, unless one workgroup sorts them alone (8192) or less than half remain
@pytest.mark.parametrize("kept,loops", [(8192, 5), (8193, 0), (8193, 8192), (8193, 8194), (8193, 8195), (8193, 60000), (40961, 1000),
                                        (196608, 12345), (196609, 100000), (3145729, 77)])
def test_sort_leaves_self_loops_out(rama, oracle32, kept, loops):
    rng = np.random.default_rng(kept + loops)
    n = 60013
    a, b = rng.integers(0, n, kept), rng.integers(0, n - 1, kept)
    b += b >= a                                                  # no loop among these; pairs may repeat
    v = rng.integers(0, n, loops)
    order = rng.permutation(kept + loops)
    i, j = np.concatenate([a, v])[order].astype(np.int32), np.concatenate([b, v])[order].astype(np.int32)
    c = (-np.abs(rng.normal(size=i.size)) - 1e-3).astype(np.float32)
    wi, wj, wc = oracle32.canonicalise(n, i, j, c)
    got = rama.contract(n, i, j, c, repeat=1, want_diag=False)
    assert np.array_equal(np_(got["i"]), wi) and np.array_equal(np_(got["j"]), wj) and np.array_equal(np_(got["c"]), wc)


@pytest.mark.parametrize("between", [8192, 8193, 60000, 65998, 65999, 66000, 66001, 66002, 300000])
def test_contraction_leaves_inner_edges_out(rama, oracle32, between):
    """1000 cliques of 12 nodes, all attractive, become 1000 nodes: 66000 edges inside them, `between` repulsive ones across."""
    from paper_2109_01838_amd import default_params
    rng = np.random.default_rng(between)
    q = np.arange(1000)[:, None] * 12
    x, y = np.triu_indices(12, 1)
    key = np.unique(rng.integers(0, 12000, 4 * between) * 12000 + rng.integers(0, 12000, 4 * between))
    lo, hi = key // 12000, key % 12000
    key = rng.permutation(key[(lo < hi) & (lo // 12 != hi // 12)])[:between]
    i = np.concatenate([(q + x).ravel(), key // 12000]).astype(np.int32)
    j = np.concatenate([(q + y).ravel(), key % 12000]).astype(np.int32)
    c = np.concatenate([1.0 + rng.random(66000), -1.0 - rng.random(between)]).astype(np.float32)
    assert i.size == 66000 + between
    want = oracle32.contract(12000, i, j, c, repeat=1, forest_ratio=1.0)
    got = rama.contract(12000, i, j, c, params=default_params(forest_ratio=1.0), repeat=1)
    assert got["n_nodes"] == want["n_nodes"] == 1000
    assert np.array_equal(np_(got["mapping"]), want["mapping"])
    for k in ("i", "j", "c"):
        assert np.array_equal(np_(got[k]), want[k]), k
    assert np.array_equal(np_(got["diag"]), want["diag"][:1000])


# --------------------------------------------------------------------------------------------
# end to end
# --------------------------------------------------------------------------------------------
@pytest.mark.parametrize("name", list(CASES))
def test_solve_end_to_end(rama, oracle32, name):
    g = CASES[name]
    n = g["n_nodes"]
    want = oracle32.solve(n, g["i"], g["j"], g["c"])
    got = rama.solve(n, g["i"], g["j"], g["c"])
    labels = np_(got["labels"])
    assert abs(got["lower_bound"] - want["lower_bound"]) <= REL * max(1.0, abs(want["lower_bound"]))
    assert abs(got["primal"] - want["primal"]) <= 5e-3 * max(1.0, abs(want["primal"]))
    # the reported primal is the cost of the returned labels, and labels are canonical
    assert abs(oracle32.multicut_cost(g["i"], g["j"], g["c"], labels) - got["primal"]) <= 1e-6 * max(1.0, abs(got["primal"]))
    assert np.all(labels[labels] == labels) and np.all(labels <= np.arange(n))
    assert got["lower_bound"] <= got["primal"] + 1e-6 * max(1.0, abs(got["primal"]))
    assert got["n_cycles_first"] == want["n_cycles_first"]
    assert got["n_edges_aug_first"] == want["n_edges_aug_first"]
    print(name, "labels identical:", bool(np.array_equal(labels, want["labels"])), "rounds", got["rounds"],
          want["rounds"], "primal", got["primal"], want["primal"], "LB", got["lower_bound"], want["lower_bound"])


@pytest.mark.parametrize("variant", ["P", "PD+", "D", "PD-matching-only", "PD-forest-always", "PD-shortest",
                                     "PD-7-then-4", "PD-7-shortest", "PD-2-dual-rounds", "D-3-dual-rounds"])
def test_solver_variants(rama, oracle32, variant):
    from paper_2109_01838_amd import default_params
    g = CASES["knn_20000"]
    n = g["n_nodes"]
    kw = {"P": dict(max_cycle_len_first=0, max_cycle_len_later=0),
          "PD+": dict(max_cycle_len_later=5),
          "D": dict(max_rounds=1),
          "PD-matching-only": dict(forest_ratio=0.0),
          "PD-forest-always": dict(forest_ratio=1.0),
          "PD-shortest": dict(shortest_only=True),
          "PD-7-then-4": dict(max_cycle_len_first=7, max_cycle_len_later=4),
          "PD-7-shortest": dict(max_cycle_len_first=7, max_cycle_len_later=7, shortest_only=True),
          "PD-2-dual-rounds": dict(dual_rounds=2),
          "D-3-dual-rounds": dict(max_rounds=1, dual_rounds=3, max_cycle_len_first=4)}[variant]
    want = oracle32.solve(n, g["i"], g["j"], g["c"], **kw)
    kw = {("shortest_cycles_only" if key == "shortest_only" else key): int(v) if key == "shortest_only" else v
          for key, v in kw.items()}
    got = rama.solve(n, g["i"], g["j"], g["c"], default_params(**kw))
    assert got["n_cycles_first"] == want["n_cycles_first"]
    print(variant, "cycles", got["n_cycles_first"], "labels identical:", bool(np.array_equal(np_(got["labels"]), want["labels"])),
          "primal", got["primal"], want["primal"], "LB", got["lower_bound"], want["lower_bound"])
    assert abs(got["lower_bound"] - want["lower_bound"]) <= REL * max(1.0, abs(want["lower_bound"]))
    assert abs(got["primal"] - want["primal"]) <= 5e-3 * max(1.0, abs(want["primal"]))


@pytest.mark.parametrize("kind,n_tri", [("apart", 1), ("apart", 2047), ("apart", 2048), ("apart", 2049), ("fan", 2048), ("fan", 2049),
                                        ("fan", 6000), ("fans", 1800), ("random", 0), ("wide", 0), ("grid", 0)])
def test_triangle_rounds_match_the_cycle_lists(rama, kind, n_tri):
    """Rounds that separate triangles only take them from the edge list itself, and one workgroup passes the messages of up
    to 2048 of them; with another cycle search than the default they go through lists of cycles.  Same integers, same sums
    in the same order: nothing may differ."""
    from paper_2109_01838_amd import default_params
    rng = np.random.default_rng(n_tri + 17)
    tau = 0.0
    if kind == "grid":
        g = inputs.cfg2(seed=3, h=220, w=221, n_seeds=30)      # 2^18 edges and more
        n, i, j, c = g["n_nodes"], g["i"], g["j"], g["c"]
    elif kind == "random":
        g = signed(inputs.random_graph(9000, 60000, 5), 6, 0.8)
        n, i, j, c = g["n_nodes"], g["i"], g["j"], g["c"]
    elif kind == "wide":       # few triangles among many edges of few nodes' each: a second round of wide tiles
        g = signed(inputs.random_graph(200000, 600000, 5), 6, 0.8)
        n, i, j, c = g["n_nodes"], g["i"], g["j"], g["c"]
    else:      # the first round joins the heavy pairs at the end and nothing else; the triangles meet the second round
        if kind == "apart":
            t = np.arange(n_tri) * 3
            tri = [(t, t + 1), (t, t + 2), (t + 1, t + 2)]
            used = 3 * n_tri
        else:      # triangles around shared repulsive edges (one, or a hundred)
            hubs = 1 if kind == "fan" else 100
            h = np.arange(n_tri) % hubs
            x = 2 * hubs + np.arange(n_tri)
            tri = [(2 * np.arange(hubs), 2 * np.arange(hubs) + 1), (2 * h, x), (2 * h + 1, x)]
            used = 2 * hubs + n_tri
        signs = rng.integers(0, 3, size=n_tri) if kind == "apart" else None
        i = np.concatenate([a for a, _ in tri])
        j = np.concatenate([b for _, b in tri])
        c = rng.uniform(0.5, 1.5, size=i.size)
        if kind == "apart":
            for k in range(3):
                c[k * n_tri:(k + 1) * n_tri][signs == k] *= -1
        else:
            c[:tri[0][0].size] *= -1
        base, tau = max(used, 6200), 2.0      # too many nodes for the rounds in one workgroup
        pairs = base + 2 * np.arange(3000)
        i = np.concatenate([i, pairs]).astype(np.int32)
        j = np.concatenate([j, pairs + 1]).astype(np.int32)
        c = np.concatenate([c, np.full(3000, 100.0)]).astype(np.float32)
        n = int(pairs[-1]) + 2
    for kw in (dict(max_cycle_len_first=0), dict(max_cycle_len_first=3, mp_iters_first=3)):
        P = default_params(contract_threshold=tau, forest_ratio=0.0, **kw)
        out = []
        for mode in (0, 1):
            rama.set_cycle_search(mode)
            got = rama.solve(n, i, j, c, P)
            out.append((np_(got["labels"]), got["primal"], got["lower_bound"],
                        [{k: v for k, v in r.items() if k not in ("ms", "workspace_peak")} for r in rama.round_stats()]))
        rama.set_cycle_search(0)
        assert np.array_equal(out[0][0], out[1][0]) and out[0][1:] == out[1][1:]
        if n_tri and kw["max_cycle_len_first"] == 0:
            assert out[0][3][1]["n_triangles"] == n_tri
        if n_tri and kw["max_cycle_len_first"] == 3:
            assert out[0][3][0]["n_triangles"] == n_tri
        if kind == "wide" and kw["max_cycle_len_first"] == 3:
            r = out[0][3][1]
            assert 1 << 18 <= r["n_edges"] <= 6 * r["n_nodes"] and 0 < r["n_triangles"] <= 2048


def separation_ms(rama, n, i, j, c, params):
    """Best of four: per round (edges, ms of separation and message passing) by the default search and through the lists of
    cycles; the two agree in every result."""
    import torch
    i, j, c = (torch.as_tensor(x).cuda() for x in (i, j, c))
    out = []
    for mode in (0, 1):
        rama.set_cycle_search(mode)
        for k in range(4):
            got = rama.solve(n, i, j, c, params)
            stats = rama.round_stats()
            ms = [r["ms"]["cycles"] + r["ms"]["dual"] for r in stats]
            best = ms if k == 0 else [min(a, b) for a, b in zip(best, ms)]
        seen = [{k: v for k, v in r.items() if k not in ("ms", "workspace_peak")} for r in stats]
        out.append((np_(got["labels"]), got["primal"], got["lower_bound"], seen, best))
    rama.set_cycle_search(0)
    assert np.array_equal(out[0][0], out[1][0]) and out[0][1:4] == out[1][1:4]
    return [(r["n_edges"], a, b) for r, a, b in zip(out[0][3], out[0][4], out[1][4])]


@pytest.mark.parametrize("pos", [0.0, 1.0])
def test_rounds_of_one_sign_are_not_searched(rama, pos):
    """Without an attractive or without a repulsive edge there is no triangle: nobody looks for one, neither behind a round
    of many triangles nor behind one of few (a search of these rows takes 0.6 to 3 ms)."""
    from paper_2109_01838_amd import default_params
    g = signed(inputs.random_graph(3000, 600000, 11), 12, pos)
    rounds = separation_ms(rama, g["n_nodes"], g["i"], g["j"], g["c"], default_params(max_cycle_len_first=3))
    for edges, ms, ms_lists in rounds:
        if edges > 20000:
            assert ms <= 3.0 * ms_lists + 0.1, rounds


@pytest.mark.parametrize("first,shape", [(0, (112, 120, 128)), (3, (1, 1500, 1600))])
def test_rounds_of_many_triangles_behind_none(rama, first, shape):
    """The round in front has no triangles, because it looks for none (first = 0) or because a grid has none: the next one's
    are far too many for one workgroup."""
    from paper_2109_01838_amd import default_params
    ids = np.arange(np.prod(shape), dtype=np.int32).reshape(shape)
    i = np.concatenate([np.delete(ids, -1, a).ravel() for a in range(3)])
    j = np.concatenate([np.delete(ids, 0, a).ravel() for a in range(3)])
    c = np.random.default_rng(3).normal(0.15, 0.5, i.size).astype(np.float32)
    rounds = separation_ms(rama, ids.size, i, j, c, default_params(max_cycle_len_first=first, max_rounds=3))
    assert rama.round_stats()[0]["n_triangles"] == 0 and rama.round_stats()[1]["n_triangles"] > 300000
    for edges, ms, ms_lists in rounds[1:]:
        assert ms <= 1.5 * ms_lists + 0.1, rounds


@pytest.mark.parametrize("kind,n,m", [("clique", 2000, 0.0), ("clique", 2000, 0.02), ("random", 3000, 600000), ("random", 20000, 500000),
                                      # a sample of all edges and of one edge less; few and many tries in all
                                      ("random", 1000, 65536), ("random", 1000, 65537), ("random", 3000, 65535), ("random", 1000, 130001)])
def test_dense_rounds_go_through_the_cycle_lists(rama, kind, n, m):
    """Where every edge has many neighbours the walk over the edge list would try far more than can be a triangle (33 ms
    instead of 2 for 2000 nodes, all joined, in clusters of ten with two edges in a hundred turned round)."""
    from paper_2109_01838_amd import default_params
    if kind == "clique":
        rng = np.random.default_rng(5)
        i, j = np.triu_indices(n, 1)
        c = np.where(i // 10 == j // 10, 1, -1) * np.where(rng.random(i.size) < m, -1, 1) * (np.abs(rng.normal(1, 0.3, i.size)) + 0.05)
        i, j, c = i.astype(np.int32), j.astype(np.int32), c.astype(np.float32)
    else:
        g = signed(inputs.random_graph(n, m, 13), 14, 0.5)
        i, j, c = g["i"], g["j"], g["c"]
    for edges, ms, ms_lists in separation_ms(rama, n, i, j, c, default_params(max_cycle_len_first=3)):
        assert edges <= 20000 or ms <= 1.5 * ms_lists + 0.1


def test_determinism(rama):
    g = CASES["knn_20000"]
    n = g["n_nodes"]
    a = rama.solve(n, g["i"], g["j"], g["c"])
    b = rama.solve(n, g["i"], g["j"], g["c"])
    assert np.array_equal(np_(a["labels"]), np_(b["labels"]))
    assert a["primal"] == b["primal"] and a["lower_bound"] == b["lower_bound"]
    c1 = rama.find_conflicted_cycles(n, g["i"], g["j"], g["c"], 5)
    m1 = rama.message_passing(n, g["i"], g["j"], g["c"], c1, 4)
    m2 = rama.message_passing(n, g["i"], g["j"], g["c"], c1, 4)
    assert np.array_equal(np_(m1["c"]), np_(m2["c"])) and m1["lower_bound"] == m2["lower_bound"]


def test_degenerate_inputs(rama):
    from paper_2109_01838_amd import RamaError, binding
    e32, ef = np.zeros(0, np.int32), np.zeros(0, np.float32)
    r = rama.solve(4, e32, e32, ef)
    assert np_(r["labels"]).tolist() == [0, 1, 2, 3] and r["primal"] == 0.0 and r["lower_bound"] == 0.0
    i, j = np.array([0, 1], np.int32), np.array([1, 2], np.int32)
    r = rama.solve(3, i, j, np.array([-1.0, -2.0], np.float32))
    assert np_(r["labels"]).tolist() == [0, 1, 2] and r["primal"] == -3.0 and r["lower_bound"] == -3.0
    r = rama.solve(3, i, j, np.array([1.0, 2.0], np.float32))
    assert np_(r["labels"]).tolist() == [0, 0, 0] and r["primal"] == 0.0
    # no nodes at all
    r = rama.solve(0, e32, e32, ef)
    assert r["labels"].numel() == 0 and r["primal"] == 0.0 and r["n_clusters"] == 0
    r = rama.contract(0, e32, e32, ef)
    assert r["n_nodes"] == 0 and r["i"].numel() == 0
    # only self-loops
    r = rama.solve(2, np.array([0, 1], np.int32), np.array([0, 1], np.int32), np.array([1.0, -1.0], np.float32))
    assert np_(r["labels"]).tolist() == [0, 1]
    cyc = rama.find_conflicted_cycles(3, i, j, np.array([1.0, 2.0], np.float32), 5)
    assert [x.shape[0] for x in cyc] == [0, 0, 0]
    with pytest.raises(RamaError) as ei:
        rama.solve(3, i, np.array([1, 3], np.int32), np.array([1.0, 1.0], np.float32))
    assert ei.value.status == binding.RAMA_ERR_BAD_GRAPH
    with pytest.raises(RamaError) as ei:
        rama.solve(3, i, j, np.array([1.0, np.inf], np.float32))
    assert ei.value.status == binding.RAMA_ERR_BAD_GRAPH
    # the context stays usable after an error
    r = rama.solve(3, i, j, np.array([1.0, 2.0], np.float32))
    assert np_(r["labels"]).tolist() == [0, 0, 0]


def test_profile_hooks_and_workspace(rama):
    g = CASES["grid3d_24"]
    rama.profile_enable(True)
    rama.solve(g["n_nodes"], g["i"], g["j"], g["c"])
    first = {k["name"] for k in rama.profile_get()}
    rama.set_cycle_search(1)       # rounds that separate triangles only through the lists of cycles as well
    rama.solve(g["n_nodes"], g["i"], g["j"], g["c"])
    rama.set_cycle_search(0)
    prof = rama.profile_get()
    rama.profile_enable(False)
    names = {k["name"] for k in prof}
    assert "k_triangles<count>" in first and not any(n.endswith("_cycles<3>") for n in first)
    assert {"k_triangle_update", "k_edge_update<false>", "k_edge_update<true>", "k_count_cycles<5>", "k_count_cycles<3>", "k_scan_emit<PackCands>", "k_reduce_runs"} <= names
    assert any(n.startswith("k_rs_scatter<") for n in names) and any(n.startswith("k_scan_apply<") for n in names)
    for k in prof:
        assert k["launches"] > 0 and k["ms"] >= 0.0 and k["bytes"] >= 0.0
    # a name filter restricts the timers
    rama.profile_enable(True, only="k_rs_scatter")
    rama.solve(g["n_nodes"], g["i"], g["j"], g["c"])
    only = rama.profile_get()
    rama.profile_enable(False)
    assert only and all(k["name"].startswith("k_rs_scatter") for k in only)
    assert rama.workspace_bytes() > 0


def test_random_sweep_of_small_instances_and_parameters(rama, oracle32):
    """Seeded sweep: small random / grid instances with random solver parameters (cycle lengths,
    iteration counts, forest switch, round limit, dual rounds, shortest-only) and a random choice of the
    cycle search (0..3) and of the entry point (rama_solve / rama_solve_static).  Labels, cycle counts,
    rounds and bounds must agree with the oracle on every one.  (Such a sweep found a rooting loop
    that gave up one check too early on trees about as deep as the graph has nodes.)"""
    from paper_2109_01838_amd import default_params
    rng = np.random.default_rng(7)
    mode_rng = np.random.default_rng(8)   # a stream of its own: the instances stay the ones of earlier versions of this test
    bad = []
    for it in range(160):
        kind = int(rng.integers(0, 4))
        seed = int(rng.integers(0, 1 << 30))
        if kind == 0:
            g = inputs.random_graph(int(rng.integers(2, 60)), int(rng.integers(1, 400)), seed, allow_messy=bool(rng.integers(0, 2)))
        elif kind == 1:
            n = int(rng.integers(50, 2000))
            g = inputs.random_graph(n, int(n * rng.uniform(1.0, 3.0)), seed)
            g = signed(g, seed, float(rng.uniform(0.5, 0.95)))
        elif kind == 2:
            g = inputs.cfg5_crop(int(rng.integers(3, 12)), seed=seed % 1000)
        else:
            g = inputs.cfg2(seed=seed % 1000, h=int(rng.integers(10, 30)), w=int(rng.integers(10, 30)), n_seeds=int(rng.integers(2, 12)))
        n = g["n_nodes"]
        shortest = bool(rng.integers(0, 2))
        kw = dict(max_cycle_len_first=int(rng.choice([0, 3, 4, 5, 6])), max_cycle_len_later=int(rng.choice([0, 3, 4])),
                  mp_iters_first=int(rng.integers(0, 8)), mp_iters_later=int(rng.integers(0, 5)),
                  forest_ratio=float(rng.choice([0.0, 0.1, 0.5, 1.0])), max_rounds=int(rng.choice([0, 0, 0, 1, 2, 3])),
                  dual_rounds=int(rng.choice([1, 1, 2, 3])))
        if kw["dual_rounds"] > 1 or (kind == 3 and not shortest):   # keeps the oracle's enumeration in seconds
            kw["max_cycle_len_first"] = min(kw["max_cycle_len_first"], 4 if kw["dual_rounds"] > 1 else 5)
            kw["max_cycle_len_later"] = min(kw["max_cycle_len_later"], 3)
        want = oracle32.solve(n, g["i"], g["j"], g["c"], shortest_only=shortest, **kw)
        rama.set_cycle_search(int(mode_rng.integers(0, 4)))
        got = rama.solve(n, g["i"], g["j"], g["c"], default_params(shortest_cycles_only=int(shortest), **kw),
                         static=bool(mode_rng.integers(0, 3) == 0))
        rama.set_cycle_search(0)
        ok = (np.array_equal(np_(got["labels"]), want["labels"]) and got["n_cycles_first"] == want["n_cycles_first"]
              and got["rounds"] == want["rounds"]
              and abs(got["lower_bound"] - want["lower_bound"]) <= REL * max(1.0, abs(want["lower_bound"]))
              and abs(got["primal"] - want["primal"]) <= 5e-3 * max(1.0, abs(want["primal"])))
        if not ok:
            bad.append((it, kind, seed, n, kw, shortest))
    assert not bad, bad


# --------------------------------------------------------------------------------------------
# the split sort (top-bit passes + one in-LDS sort) is the same stable sort as passes over all bits
# --------------------------------------------------------------------------------------------
@pytest.fixture(scope="module")
def rama_split():
    from paper_2109_01838_amd import Rama
    r = Rama("cuda:0")
    r.set_sort_split(0, 0)          # every sort of two or more elements takes the split path
    yield r
    r.close()


def star_graph(n_leaves, seed):
    """Node 0 joined to every other node, plus a sparse ring: all edges of the hub share their
    first endpoint, so the hub's segment exceeds what a workgroup can sort in LDS."""
    rng = np.random.default_rng(seed)
    leaves = np.arange(1, n_leaves + 1, dtype=np.int32)
    i = np.concatenate([np.zeros(n_leaves, np.int32), leaves[:-1]])
    j = np.concatenate([leaves, leaves[1:]])
    mag = np.abs(rng.normal(0.0, 1.0, i.size)).astype(np.float32) + 0.05
    c = np.where(rng.random(i.size) < 0.7, mag, -mag).astype(np.float32)
    perm = rng.permutation(i.size)
    return dict(name=f"star_{n_leaves}", n_nodes=n_leaves + 1, i=i[perm], j=j[perm], c=c[perm])


def gappy_graph(n, kind, seed):
    """Graphs whose node rows have long empty stretches.  'clusters': dense little cliques-with-noise far apart
    in the node numbering (many edges, gaps of thousands of rows between them); 'sparse': a few triangles
    scattered over many nodes (far fewer edges than rows); 'tail': all edges among the last few nodes."""
    rng = np.random.default_rng(seed)
    ii, jj = [], []
    if kind == "clusters":
        for base in range(0, n - 64, max(64, n // 40)):
            nodes = base + np.arange(48)
            a = rng.choice(nodes, 400); b = rng.choice(nodes, 400)
            ii.append(a); jj.append(b)
    elif kind == "sparse":
        for base in rng.choice(n - 3, 60, replace=False):
            ii.append(np.array([base, base + 1, base])); jj.append(np.array([base + 1, base + 2, base + 2]))
    else:
        nodes = n - 40 + np.arange(40)
        ii.append(rng.choice(nodes, 500)); jj.append(rng.choice(nodes, 500))
    i = np.concatenate(ii).astype(np.int32); j = np.concatenate(jj).astype(np.int32)
    keep = i != j
    i, j = i[keep], j[keep]
    mag = np.abs(rng.normal(0.0, 1.0, i.size)).astype(np.float32) + 0.05
    c = np.where(rng.random(i.size) < 0.65, mag, -mag).astype(np.float32)
    return dict(n_nodes=n, i=i, j=j, c=c)


@pytest.mark.parametrize("kind", ["clusters", "sparse", "tail"])
@pytest.mark.parametrize("n", [5000, 60000, 300000])
def test_rows_with_long_empty_stretches(rama, oracle32, kind, n):
    """Row pointers over node sets that are mostly empty: long gaps are filled by whole workgroups, sparse key
    sets are searched per row; cycles, message passing and the whole solve must not notice."""
    g = gappy_graph(n, kind, 11)
    want = oracle32.find_conflicted_cycles(n, g["i"], g["j"], g["c"], 5)
    got = rama.find_conflicted_cycles(n, g["i"], g["j"], g["c"], 5)
    for a, b in zip(got, want):
        assert np.array_equal(np_(a), b)
    wmp = oracle32.message_passing(n, g["i"], g["j"], g["c"], want, 3)
    mp = rama.message_passing(n, g["i"], g["j"], g["c"], want, 3)
    assert np.array_equal(np_(mp["i"]), wmp["i"]) and np.array_equal(np_(mp["j"]), wmp["j"])
    assert rel_close(np_(mp["c"]), wmp["c"])
    ws = oracle32.solve(n, g["i"], g["j"], g["c"])
    gs = rama.solve(n, g["i"], g["j"], g["c"])
    assert gs["n_cycles_first"] == ws["n_cycles_first"] and gs["rounds"] == ws["rounds"]
    assert np.array_equal(np_(gs["labels"]), ws["labels"])
    assert abs(gs["lower_bound"] - ws["lower_bound"]) <= REL * max(1.0, abs(ws["lower_bound"]))
    print(kind, n, [x.shape[0] for x in want], gs["rounds"])


@pytest.mark.parametrize("name", list(CASES))
def test_split_sort_stagewise(rama_split, oracle32, name):
    from paper_2109_01838_amd import default_params
    g = CASES[name]
    n = g["n_nodes"]
    lmax = 4 if name == "random_dense" else 5
    cyc = oracle32.find_conflicted_cycles(n, g["i"], g["j"], g["c"], lmax)
    got = rama_split.find_conflicted_cycles(n, g["i"], g["j"], g["c"], lmax)
    for a, b in zip(got, cyc):
        assert np.array_equal(np_(a), b)
    want = oracle32.message_passing(n, g["i"], g["j"], g["c"], cyc, 3)
    mp = rama_split.message_passing(n, g["i"], g["j"], g["c"], cyc, 3)
    assert np.array_equal(np_(mp["i"]), want["i"]) and np.array_equal(np_(mp["j"]), want["j"])
    assert rel_close(np_(mp["c"]), want["c"])
    for forest_ratio in (0.1, 1.0):
        w = oracle32.contract(n, want["i"], want["j"], want["c"], forest_ratio=forest_ratio)
        con = rama_split.contract(n, want["i"], want["j"], want["c"], params=default_params(forest_ratio=forest_ratio))
        assert np.array_equal(np_(con["mapping"]), w["mapping"])
        assert np.array_equal(np_(con["i"]), w["i"]) and np.array_equal(np_(con["j"]), w["j"])
        assert rel_close(np_(con["c"]), w["c"])


@pytest.mark.parametrize("name", list(CASES) + ["hubs", "star_9", "star_40000"])
def test_split_sort_solve(rama, rama_split, oracle32, name):
    """Same labels, bounds and counts from both sort paths (bit for bit: both are the same stable
    sort), and both agree with the oracle.  star_40000 holds a segment no workgroup can take, which
    sends the split path back to passes over all bits after its top-bit passes."""
    g = CASES[name] if name in CASES else (inputs.hub_graph() if name == "hubs" else star_graph(int(name[5:]), 3))
    n = g["n_nodes"]
    a = rama.solve(n, g["i"], g["j"], g["c"])
    b = rama_split.solve(n, g["i"], g["j"], g["c"])
    want = oracle32.solve(n, g["i"], g["j"], g["c"])
    assert np.array_equal(np_(a["labels"]), np_(b["labels"]))
    assert a["primal"] == b["primal"] and a["lower_bound"] == b["lower_bound"]
    assert a["n_cycles_first"] == b["n_cycles_first"] == want["n_cycles_first"]
    assert a["rounds"] == b["rounds"]
    assert np.array_equal(np_(b["labels"]), want["labels"])
    assert abs(b["lower_bound"] - want["lower_bound"]) <= REL * max(1.0, abs(want["lower_bound"]))


def test_split_sort_takes_its_kernels(rama_split):
    g = CASES["knn_20000"]
    rama_split.profile_enable(True)
    rama_split.solve(g["n_nodes"], g["i"], g["j"], g["c"])
    names = {k["name"] for k in rama_split.profile_get()}
    rama_split.profile_enable(False)
    assert "k_seg_bounds" in names and "k_rs_local<u64,u32>" in names and "k_rs_local<u32,u32>" in names


def test_split_sort_with_wide_local_keys(rama_split, oracle32):
    """Few edges over many nodes: one pass over the top bits leaves more than 26 low bits, which do
    not fit the 32-bit keys of the in-LDS sort, so its 64-bit variant runs."""
    from paper_2109_01838_amd import default_params
    g = signed(inputs.random_graph(200000, 400000, 21), 21, 0.75)
    perm = np.random.default_rng(5).permutation(g["i"].size)     # unsorted input: canonicalising it sorts (key, cost) pairs
    g = dict(g, i=g["i"][perm], j=g["j"][perm], c=g["c"][perm])
    n = g["n_nodes"]
    rama_split.profile_enable(True)
    got = rama_split.solve(n, g["i"], g["j"], g["c"])
    names = {k["name"] for k in rama_split.profile_get()}
    rama_split.profile_enable(False)
    assert {"k_rs_local<u64,u32,wide>", "k_rs_local<u64,wide>"} <= names
    want = oracle32.solve(n, g["i"], g["j"], g["c"])
    assert np.array_equal(np_(got["labels"]), want["labels"])
    assert got["n_cycles_first"] == want["n_cycles_first"] and got["rounds"] == want["rounds"]
    assert abs(got["lower_bound"] - want["lower_bound"]) <= REL * max(1.0, abs(want["lower_bound"]))
    for forest_ratio in (0.1, 1.0):
        w = oracle32.contract(n, g["i"], g["j"], g["c"], forest_ratio=forest_ratio)
        con = rama_split.contract(n, g["i"], g["j"], g["c"], params=default_params(forest_ratio=forest_ratio))
        assert np.array_equal(np_(con["mapping"]), w["mapping"])
        assert np.array_equal(np_(con["i"]), w["i"]) and np.array_equal(np_(con["j"]), w["j"])
        assert rel_close(np_(con["c"]), w["c"])


def test_context_on_a_side_stream_and_two_contexts(rama):
    """A context bound to a non-default stream (default priority) gives the same result as the
    default-stream context, also when the two are used in turn."""
    import torch
    from paper_2109_01838_amd import Rama
    g = CASES["grid3d_24"]
    n = g["n_nodes"]
    base = rama.solve(n, g["i"], g["j"], g["c"])
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        other = Rama("cuda:0")
        assert other.stream.cuda_stream == side.cuda_stream and other.stream.cuda_stream != rama.stream.cuda_stream
        a = other.solve(n, g["i"], g["j"], g["c"])
        cyc = other.find_conflicted_cycles(n, g["i"], g["j"], g["c"], 5)
    side.synchronize()
    b = rama.solve(n, g["i"], g["j"], g["c"])
    with torch.cuda.stream(side):
        a2 = other.solve(n, g["i"], g["j"], g["c"])
    side.synchronize()
    for r in (a, b, a2):
        assert np.array_equal(np_(r["labels"]), np_(base["labels"])) and r["primal"] == base["primal"]
        assert r["lower_bound"] == base["lower_bound"]
    want = rama.find_conflicted_cycles(n, g["i"], g["j"], g["c"], 5)
    assert all(np.array_equal(np_(x), np_(y)) for x, y in zip(cyc, want))
    other.close()


# --------------------------------------------------------------------------------------------
# workspace allocator callbacks and per-round records
# --------------------------------------------------------------------------------------------
@pytest.mark.parametrize("ratio", [0.0, 1.0], ids=["matching", "forest"])
def test_contraction_holds_no_memory_of_the_matching(rama, ratio):
    """What a round without separation needs at most: the matching its candidates twice (2 * 16 bytes), mates and three rank
    words per node; the contraction relabelled keys, the sort's two pairs and its table, mates and mapping -- and not the
    candidates.  An eighth of a byte per edge and 64 KiB are allowed for scan plans and counters."""
    from paper_2109_01838_amd import default_params
    g = inputs.cfg2(h=100, w=100, n_seeds=33)
    n, m, na = g["n_nodes"], g["i"].size, int((g["c"] > 0).sum())
    rama.solve(n, g["i"], g["j"], g["c"], static=True,
               params=default_params(max_cycle_len_first=0, max_cycle_len_later=0, forest_ratio=ratio, max_rounds=1))
    most = max(12 * m + 32 * na + 28 * n, 12 * m + 8 * m + 12 * m + 4 * m + m + 8 * n)
    assert rama.round_stats()[0]["workspace_peak"] <= most + m // 8 + (1 << 16)


@pytest.mark.parametrize("background", [8770, 8840, 8900, 9225])
def test_static_workspace_near_its_limit(rama, background):
    """Hubs whose triangles fill the static workspace to nine tenths and more: every one of these solves has to find room."""
    from paper_2109_01838_amd import default_params
    g = inputs.hub_graph(n_nodes=4000, hubs=(0, 1000, 2000, 3000), hub_degree=700, n_background=background)
    params = default_params(max_rounds=4)
    want = rama.solve(g["n_nodes"], g["i"], g["j"], g["c"], params=params)
    got = rama.solve(g["n_nodes"], g["i"], g["j"], g["c"], params=params, static=True)
    assert got["lower_bound"] == want["lower_bound"] and np.array_equal(np_(got["labels"]), np_(want["labels"]))


def test_runs_with_a_repeated_pair_hold_no_memory_of_the_attempt(rama):
    """Three sorted runs whose last edge repeats a pair of the first: interleaving gives up, and the merge that follows needs
    two key and two cost arrays (24 bytes per edge) beside what the pool keeps of the attempt, of which the costs take
    8.  (With the attempt's 12 bytes per edge held it took 36.)"""
    import torch
    from paper_2109_01838_amd import Rama
    s = 100
    v = np.arange(s ** 3, dtype=np.int32).reshape(s, s, s)
    i = np.concatenate([v[:-1].ravel(), v[:, :-1].ravel(), v[:, :, :-1].ravel(), v[-2:-1, -1, -1].ravel()])
    j = np.concatenate([v[1:].ravel(), v[:, 1:].ravel(), v[:, :, 1:].ravel(), v[-1:, -1, -1].ravel()])
    m = i.size
    d = [torch.as_tensor(x).cuda() for x in (i, j, np.ones(m, np.float32))]
    fresh = Rama("cuda:0", allocator="hip")
    before = fresh.workspace_bytes()
    assert fresh.find_conflicted_cycles(s ** 3, *d, 3)[0].shape[0] == 0
    assert fresh.workspace_bytes() - before < 31 * m, (fresh.workspace_bytes() - before) / m
    fresh.close()


@pytest.mark.parametrize("pos,through_lists", [(0.05, True), (0.075, False)])
def test_static_workspace_of_a_dense_graph(rama, pos, through_lists):
    """Where the static workspace has no room for the lists of cycles a dense graph's triangles come from its edges."""
    from paper_2109_01838_amd import default_params
    i, j = (x.astype(np.int32) for x in np.triu_indices(724, 1))
    rng = np.random.default_rng(75)
    c = ((rng.random(i.size) + 0.05) * np.where(rng.random(i.size) < pos, 1, -1)).astype(np.float32)
    params = default_params(max_cycle_len_first=3)
    want = rama.solve(724, i, j, c, params)
    got = rama.solve(724, i, j, c, params, static=True)
    assert rama.round_stats()[0]["n_triangles"] == want["n_triangles_first"] > 400000
    # 70 to 75 bytes per triangle, against 58
    assert (want["n_triangles_first"] * 75 < 64 << 20) == through_lists and (want["n_triangles_first"] * 70 > 64 << 20) == (not through_lists)
    assert np.array_equal(np_(got["labels"]), np_(want["labels"]))
    assert (got["primal"], got["lower_bound"], got["rounds"]) == (want["primal"], want["lower_bound"], want["rounds"])


@pytest.mark.parametrize("points", [60800, 60000])
def test_static_workspace_near_its_limit_with_kept_triangles(rama, points):
    from paper_2109_01838_amd import default_params
    g = inputs.cfg3(n_points=points, n_seeds=points // 200)
    params = default_params(max_rounds=2, dual_rounds=2)
    want = rama.solve(g["n_nodes"], g["i"], g["j"], g["c"], params=params)
    got = rama.solve(g["n_nodes"], g["i"], g["j"], g["c"], params=params, static=True)
    assert got["lower_bound"] == want["lower_bound"] and np.array_equal(np_(got["labels"]), np_(want["labels"]))


def test_allocator_callbacks_and_injected_out_of_memory(rama):
    """The workspace comes from the caller's allocator; an allocator that runs dry at its n-th call makes the
    call in progress end with RAMA_ERR_OOM, everything taken so far goes back, and the ctx stays usable."""
    import torch
    from paper_2109_01838_amd import Rama, RamaError, binding
    g = CASES["grid3d_24"]
    n = g["n_nodes"]
    base = rama.solve(n, g["i"], g["j"], g["c"])
    live, calls, fail_from = {}, [0], [None]

    def alloc(nbytes):
        calls[0] += 1
        if fail_from[0] is not None and calls[0] >= fail_from[0]:
            return None
        p = torch.cuda.caching_allocator_alloc(int(nbytes), 0)
        live[p] = nbytes
        return p

    def free(ptr):
        assert ptr in live
        del live[ptr]
        torch.cuda.caching_allocator_delete(ptr)

    r = Rama("cuda:0", allocator=(alloc, free))
    at_create = calls[0]                             # the ctx's own few words
    a = r.solve(n, g["i"], g["j"], g["c"])
    assert np.array_equal(np_(a["labels"]), np_(base["labels"])) and a["primal"] == base["primal"]
    total_calls = calls[0] - at_create               # allocator calls of one solve on a fresh ctx
    assert total_calls > 5 and len(live) > 0 and sum(live.values()) == r.workspace_bytes()
    r.close()
    assert not live                                  # every block went back through the callback
    for k in (1, 3, total_calls // 2, total_calls):
        r = Rama("cuda:0", allocator=(alloc, free))
        calls[0], fail_from[0] = 0, k
        with pytest.raises(RamaError) as ei:
            r.solve(n, g["i"], g["j"], g["c"])
        assert ei.value.status == binding.RAMA_ERR_OOM, ei.value
        assert sum(live.values()) == r.workspace_bytes()   # what was in use at the failure is cached, nothing is lost
        fail_from[0] = None
        b = r.solve(n, g["i"], g["j"], g["c"])       # same ctx, allocator working again
        assert np.array_equal(np_(b["labels"]), np_(base["labels"])) and b["lower_bound"] == base["lower_bound"]
        r.close()
        assert not live
    # the library's own hipMalloc path still exists
    r = Rama("cuda:0", allocator="hip")
    c = r.solve(n, g["i"], g["j"], g["c"])
    assert np.array_equal(np_(c["labels"]), np_(base["labels"]))
    r.close()


def test_triangles_of_long_rows_need_no_more_memory(oracle32):
    """Sixteen lanes an edge note the common neighbours that they count in memory that the call has done with.  Whatever the
    caller's allocator can give to the workspace and to the results together: where the search by one thread an edge gets
    through, so does this one, with the same triangles, and no failure is left behind."""
    import torch
    from paper_2109_01838_amd import Rama, RamaError

    class Limited(Rama):
        def __init__(self, limit):
            self.out, self.peak, self.limit, sizes = 0, 0, limit, {}

            def alloc(nbytes):
                self.take(nbytes)
                p = torch.cuda.caching_allocator_alloc(int(nbytes), 0)
                sizes[p] = nbytes
                return p

            def free(p):
                self.out -= sizes.pop(p)
                torch.cuda.caching_allocator_delete(p)
            super().__init__("cuda:0", allocator=(alloc, free))

        def take(self, nbytes):
            if self.out + nbytes > self.limit:
                raise MemoryError
            self.out += nbytes
            self.peak = max(self.peak, self.out)

        def _empty(self, n, dtype):
            self.take(max(int(n), 1) * 4)
            return super()._empty(n, dtype)

    def search(g, mode, limit):
        r = Limited(limit)
        try:
            r.set_cycle_search(mode)
            try:
                tri = np_(r.find_conflicted_cycles(g["n_nodes"], g["i"], g["j"], g["c"], 3)[0])
            except (RamaError, MemoryError):
                return None, r.peak
            assert r.lib.rama_last_error(r.ctx) == b""
            return tri, r.peak
        finally:
            r.close()

    for h, w in ((40, 41), (130, 131), (310, 231)):       # 4e3, 4e4 and 1.7e5 repulsive edges (edges with triangles are listed from 2^17 on)
        n, i, j = inputs.grid_edges((h, w), [(0, 1), (0, 2)])
        parts = [(i, j)]
        v = np.arange(h * w, dtype=np.int32).reshape(h, w)
        for a in (1, 2):
            for b in range(-2, 3):
                parts.append((v[:h - a, max(0, -b):w - max(0, b)].ravel(), v[a:, max(0, b):w + min(0, b)].ravel()))
        i, j = (np.concatenate([p[k] for p in parts]) for k in (0, 1))
        rng = np.random.default_rng(h)
        g = dict(n_nodes=n, i=i, j=j, c=(rng.random(i.size) + 0.1).astype(np.float32) * np.where(rng.random(i.size) < 0.2, -1, 1).astype(np.float32))
        for k in "ijc":
            g[k] = torch.as_tensor(g[k]).cuda()
        want, peak = search(g, 1, 1 << 40)
        got, most = search(g, 2, 1 << 40)
        assert np.array_equal(got, want) and want.shape[0] > 10 * h * w
        assert most <= peak + (1 << 16), (most, peak)
        passed = 0
        for limit in np.linspace(0.8 * peak, peak, 21).astype(np.int64).tolist():
            want_at, _ = search(g, 1, limit)
            got_at, _ = search(g, 2, limit)
            assert got_at is not None or want_at is None, (limit, peak)
            assert got_at is None or np.array_equal(got_at, want)
            passed += want_at is not None
        assert 0 < passed
    o = oracle32.find_conflicted_cycles(*(g[k] if k == "n_nodes" else np_(g[k]) for k in ("n_nodes", "i", "j", "c")), 3)
    assert np.array_equal(want, o[0])


def test_round_records(rama, oracle32):
    g = CASES["knn_20000"]
    n = g["n_nodes"]
    got = rama.solve(n, g["i"], g["j"], g["c"])
    rounds = rama.round_stats()
    assert len(rounds) == got["rounds"] >= 2
    ic, jc, cc = oracle32.canonicalise(n, g["i"], g["j"], g["c"])
    first = rounds[0]
    assert first["n_nodes"] == n and first["n_edges"] == ic.size
    assert first["n_attractive"] == int((cc > 0).sum()) and first["n_repulsive"] == int((cc < 0).sum())
    assert first["n_cycles"] == got["n_cycles_first"] and first["n_triangles"] == got["n_triangles_first"]
    assert first["n_edges_aug"] == got["n_edges_aug_first"]
    want = oracle32.find_conflicted_cycles(n, g["i"], g["j"], g["c"], 5)
    assert first["n_cycles"][:3] == [w.shape[0] for w in want]
    for a, b in zip(rounds, rounds[1:]):
        assert b["n_nodes"] < a["n_nodes"]
        assert a["n_contracted"] > 0 and b["n_edges"] <= a["n_edges_aug"]
        if not a["used_forest"]:
            assert b["n_nodes"] == a["n_nodes"] - a["n_contracted"]     # a matching joins pairs
    assert rounds[-1]["n_contracted"] == 0
    assert all(r["workspace_peak"] > 0 for r in rounds)
    assert all(r["ms"]["cycles"] >= 0 and r["ms"]["dual"] >= 0 and r["ms"]["contract"] > 0 for r in rounds)
    s = got["ms"]
    assert abs(sum(r["ms"]["contract"] for r in rounds) - s["contract"]) < 1e-6 and s["total"] > s["contract"]
