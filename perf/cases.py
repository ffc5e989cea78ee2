"""What a user of this library has it do, as measurable cases.

Every case is one call of a public entry point of `paper_2109_01838_amd.Rama` on a synthetic multicut instance
that is in device memory already.  The instances follow the recipes of `paper_2109_01838_amd/inputs.py` (planted
clusters, fp32 costs, sign flips), drawn on the GPU so that a fresh seed costs a moment and not minutes:

  grid4       2-D 4-connected grid, 8x8 blocks: superpixel-sized, every call is launches and waits
  longrange   2-D grid with offsets 1, 3 and 9 (image segmentation with long-range affinities)
  window      2-D grid, every pixel joined to its 5x5 window: dense rows, many triangles, like contracted graphs
  knn         random points joined to their 6 nearest neighbours (irregular, superpixel-graph-like; 3-, 4-, 5-cycles)
  grid3d      3-D 6-connected voxel grid (volume segmentation)

Edge lists come in the order a program makes them in: grids direction by direction, neighbour graphs sorted, and
`shuffled` in arbitrary order and orientation with a few parallel edges (lists out of a hash map).
"""
import math

import torch

from paper_2109_01838_amd import Rama, default_params

GRAPHS_2D = {
    "grid4": ((0, 1), (1, 0)),
    "longrange": ((0, 1), (1, 0), (0, 3), (3, 0), (0, 9), (9, 0)),
    "window": tuple((a, b) for a in range(3) for b in range(-2, 3) if a > 0 or b > 0),
}
OFFSETS_3D = ((0, 0, 1), (0, 1, 0), (1, 0, 0))
# (mean, deviation, share of flipped signs) of the costs inside a cluster; across clusters the mean is negative
COSTS = {"grid4": (1.0, 0.5, 0.0), "longrange": (0.8, 0.6, 0.05), "window": (0.8, 0.6, 0.05), "grid3d": (0.7, 0.7, 0.05)}


# ---------------------------------------------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------------------------------------------
def listed():
    return [
        # the smallest problem anybody sends: interactive use, one superpixel patch; all latency
        dict(name="solve_grid4_32", op="solve", graph="grid4", d=1, h=32, w=32, shuffled=False),
        # a serving loop that must not allocate: small tiles through the static workspace
        dict(name="static_longrange_128", op="static", graph="longrange", d=1, h=128, w=128, shuffled=False),
        # one street-scene image with long-range affinities
        dict(name="solve_longrange_512", op="solve", graph="longrange", d=1, h=512, w=512, shuffled=False),
        # a superpixel graph of a whole data set slice, irregular degrees
        dict(name="solve_knn_1000000", op="solve", graph="knn", n=1000000, shuffled=False),
        # a ragged block of a volume whose edge list comes in arbitrary order
        dict(name="solve_grid3d_61x97x131_shuffled", op="solve", graph="grid3d", d=61, h=97, w=131, shuffled=True),
        # the headline: a 320^3 volume, 9.8e7 edges
        dict(name="solve_grid3d_320", op="solve", graph="grid3d", d=320, h=320, w=320, shuffled=False),
        # separation alone (a caller with a dual solver of its own), all lengths up to 5
        dict(name="cycles_knn_300007", op="cycles", graph="knn", n=300007, shuffled=False, length=5),
        # separation on a dense graph as later rounds see it: triangles only
        dict(name="cycles_window_400x301", op="cycles", graph="window", d=1, h=400, w=301, shuffled=False, length=3),
        # message passing alone, the paper's k = 10, on the cycles of a volume
        dict(name="mp_grid3d_160", op="mp", graph="grid3d", d=160, h=160, w=160, shuffled=False, k=10),
        # one primal update with diagonal (a caller with a loop of its own)
        dict(name="contract_grid3d_127x160x161", op="contract", graph="grid3d", d=127, h=160, w=161, shuffled=False, repeat=1),
        # the purely primal solver "P": contraction until nothing attracts
        dict(name="contract_longrange_300x301", op="contract", graph="longrange", d=1, h=300, w=301, shuffled=False, repeat=0),
        # a tighter bound: separation and message passing twice on the same graph
        dict(name="dual2_longrange_180x181", op="dual", graph="longrange", d=1, h=180, w=181, shuffled=False, rounds=2),
    ]


def _between(rng, lo, hi):
    """A whole number, uniform over the logarithm of [lo, hi]."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _box(rng, lo, hi):
    """d x h x w of about lo..hi voxels, sides up to a factor of two apart."""
    side = _between(rng, lo, hi) ** (1.0 / 3.0)
    a, b = rng.uniform(0.75, 1.3), rng.uniform(0.75, 1.3)
    return dict(d=max(2, int(side * a)), h=max(2, int(side * b)), w=max(2, int(side / (a * b))))


def _sheet(rng, lo, hi):
    side = _between(rng, lo, hi) ** 0.5
    a = rng.uniform(0.7, 1.4)
    return dict(d=1, h=max(10, int(side * a)), w=max(10, int(side / a)))


def draw(rng):
    kind = rng.choice(["small", "static", "longrange", "knn", "volume", "volume", "cycles", "mp", "contract", "primal", "dual"])
    shuffled = rng.random() < 0.25
    if kind == "small":
        return dict(op="solve", graph="grid4", shuffled=shuffled, **_sheet(rng, 100, 20000))
    if kind == "static":
        return dict(op="static", graph="longrange", shuffled=shuffled, **_sheet(rng, 2000, 30000))
    if kind == "longrange":
        return dict(op="solve", graph="longrange", shuffled=shuffled, **_sheet(rng, 20000, 600000))
    if kind == "knn":
        return dict(op="solve", graph="knn", n=_between(rng, 20000, 1200000), shuffled=shuffled)
    if kind == "volume":
        return dict(op="solve", graph="grid3d", shuffled=shuffled, **_box(rng, 50000, 16000000))
    if kind == "cycles":
        graph = rng.choice(["knn", "longrange", "window"])
        if graph == "knn":
            return dict(op="cycles", graph=graph, n=_between(rng, 20000, 800000), shuffled=shuffled, length=rng.choice([3, 4, 5]))
        length = rng.choice([4, 5]) if graph == "longrange" else 3
        return dict(op="cycles", graph=graph, shuffled=shuffled, length=length, **_sheet(rng, 10000, 400000))
    if kind == "mp":
        return dict(op="mp", graph="grid3d", shuffled=shuffled, k=rng.choice([1, 5, 10]), **_box(rng, 30000, 8000000))
    if kind == "contract":
        return dict(op="contract", graph="grid3d", shuffled=shuffled, repeat=1, **_box(rng, 30000, 8000000))
    if kind == "primal":
        return dict(op="contract", graph="longrange", shuffled=shuffled, repeat=0, **_sheet(rng, 10000, 400000))
    return dict(op="dual", graph="longrange", shuffled=shuffled, rounds=rng.choice([1, 2]), **_sheet(rng, 3000, 33000))


# ---------------------------------------------------------------------------------------------------------------
# the instances
# ---------------------------------------------------------------------------------------------------------------
def _voronoi(shape, n_seeds, gen, dev):
    """Cluster of every voxel: its (nearly always) nearest of n_seeds uniform seed voxels, by jump flooding."""
    d, h, w = shape
    pos = torch.stack([torch.randint(0, s, (n_seeds,), generator=gen, device=dev) for s in shape])
    label = torch.full((d * h * w,), -1, dtype=torch.int64, device=dev)
    label.scatter_reduce_(0, (pos[0] * h + pos[1]) * w + pos[2], torch.arange(n_seeds, device=dev), "amax")
    label = label.to(torch.int32).view(d, h, w)
    at = pos.to(torch.float32)
    grid = [torch.arange(s, dtype=torch.float32, device=dev) for s in shape]
    grid = (grid[0].view(-1, 1, 1), grid[1].view(1, -1, 1), grid[2].view(1, 1, -1))

    def distance(lab, z, y, x):
        q = lab.clamp(min=0)
        r = (at[0][q] - z).square_() + (at[1][q] - y).square_() + (at[2][q] - x).square_()
        return r.masked_fill_(lab < 0, math.inf)

    spacing = (d * h * w / n_seeds) ** (1.0 / (2 if d == 1 else 3))
    step = 1 << max(0, math.ceil(math.log2(1.5 * spacing)))
    best = distance(label, *grid)
    while step >= 1:
        for a in ((0,) if d == 1 else (-step, 0, step)):
            for b in (-step, 0, step):
                for c in (-step, 0, step):
                    if (a == 0 and b == 0 and c == 0) or abs(a) >= d or abs(b) >= h or abs(c) >= w:
                        continue
                    to = tuple(slice(max(0, -k), s - max(0, k)) for k, s in zip((a, b, c), shape))
                    fro = tuple(slice(max(0, k), s - max(0, -k)) for k, s in zip((a, b, c), shape))
                    lab = label[fro].clone()
                    dist = distance(lab, grid[0][to[0]], grid[1][:, to[1]], grid[2][:, :, to[2]])
                    closer = dist < best[to]
                    best[to] = torch.where(closer, dist, best[to])
                    label[to] = torch.where(closer, lab, label[to])
        step //= 2
    return label.view(-1)


def _shape_offsets(case):
    shape = (case["d"], case["h"], case["w"])
    return shape, OFFSETS_3D if case["graph"] == "grid3d" else [(0, a, b) for a, b in GRAPHS_2D[case["graph"]]]


def _grid(shape, offsets, dev):
    """Edges x -> x + offset, one block per offset, every block in ascending source order."""
    ids = torch.arange(shape[0] * shape[1] * shape[2], dtype=torch.int32, device=dev).view(shape)
    i, j = [], []
    for off in offsets:
        if any(abs(k) >= s for k, s in zip(off, shape)):
            continue
        i.append(ids[tuple(slice(max(0, -k), s - max(0, k)) for k, s in zip(off, shape))].reshape(-1))
        j.append(ids[tuple(slice(max(0, k), s - max(0, -k)) for k, s in zip(off, shape))].reshape(-1))
    return torch.cat(i), torch.cat(j)


def _knn(n, k, gen, dev):
    """n uniform points and the canonical edge list of their k-nearest-neighbour graph (looked for in the 3x3 bins
    around a point)."""
    pts = torch.rand((n, 2), generator=gen, device=dev)
    side = max(1, int((n / 6.0) ** 0.5))
    cell = (pts * side).to(torch.int64).clamp_(max=side - 1)
    flat = cell[:, 0] * side + cell[:, 1]
    order = torch.argsort(flat, stable=True)
    count = torch.bincount(flat, minlength=side * side)
    start = torch.cumsum(count, 0) - count
    cap = int(count.max())
    bins = torch.full((side * side + 1, cap), -1, dtype=torch.int64, device=dev)     # the last bin stays empty
    where = flat[order]
    bins[where, torch.arange(n, device=dev) - start[where]] = order
    lo, hi = [], []
    for q in torch.arange(n, device=dev).split(1 << 18):
        cand = []
        for a in (-1, 0, 1):
            for b in (-1, 0, 1):
                y, x = cell[q, 0] + a, cell[q, 1] + b
                inside = (y >= 0) & (y < side) & (x >= 0) & (x < side)
                cand.append(bins[torch.where(inside, y * side + x, side * side)])
        cand = torch.cat(cand, 1)
        dist = (pts[cand.clamp(min=0)] - pts[q].unsqueeze(1)).square().sum(2)
        dist.masked_fill_((cand < 0) | (cand == q.unsqueeze(1)), math.inf)
        near = torch.topk(dist, k, largest=False)
        nb = torch.gather(cand, 1, near.indices)
        ok = torch.isfinite(near.values)
        src = q.unsqueeze(1).expand_as(nb)[ok]
        nb = nb[ok]
        lo.append(torch.minimum(src, nb))
        hi.append(torch.maximum(src, nb))
    key = torch.unique(torch.cat(lo) * n + torch.cat(hi))
    return pts, (key // n).to(torch.int32), (key % n).to(torch.int32)


def _instance(case, seed):
    """n_nodes, i, j, c on the GPU."""
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed)
    if case["graph"] == "knn":
        n = case["n"]
        pts, i, j = _knn(n, 6, gen, dev)
        # planted clusters of 200 points each on average, costs = logit of a Beta-distributed probability; the
        # Beta(5,2) and Beta(2,5) variables are the fifth and the second smallest of six uniform ones
        side = max(2, int(n ** 0.5))
        truth = _voronoi((1, side, side), max(2, n // 200), gen, dev)
        cell = (pts * side).to(torch.int64).clamp_(max=side - 1)
        truth = truth[cell[:, 0] * side + cell[:, 1]]
        u = torch.rand((i.numel(), 6), generator=gen, device=dev).sort(1).values
        p = torch.where(truth[i] == truth[j], u[:, 4], u[:, 1]).clamp_(1e-6, 1.0 - 1e-6)
        c = torch.log(p / (1.0 - p))
    else:
        shape, offsets = _shape_offsets(case)
        n = math.prod(shape)
        i, j = _grid(shape, offsets, dev)
        if case["graph"] == "grid4":
            y, x = torch.meshgrid(torch.arange(shape[1], device=dev) // 8, torch.arange(shape[2], device=dev) // 8, indexing="ij")
            truth = (y * shape[2] + x).reshape(-1)
        else:       # one cluster per 328 voxels, per 524 pixels
            truth = _voronoi(shape, max(2, n // (328 if case["graph"] == "grid3d" else 524)), gen, dev)
        mean, dev_c, flip = COSTS[case["graph"]]
        z = torch.randn(i.numel(), generator=gen, device=dev)
        c = z * dev_c + torch.where(truth[i] == truth[j], mean, -mean)
        if flip > 0.0:
            c = torch.where(torch.rand(i.numel(), generator=gen, device=dev) < flip, -c, c)
    if case["shuffled"]:        # any order, either orientation, one edge in a hundred given in two parts
        twice = torch.randint(0, i.numel(), (i.numel() // 100,), generator=gen, device=dev)
        i, j, c = torch.cat([i, j[twice]]), torch.cat([j, i[twice]]), torch.cat([c, 0.25 * c[twice]])
        perm = torch.randperm(i.numel(), generator=gen, device=dev)
        i, j, c = i[perm], j[perm], c[perm]
        swap = torch.rand(i.numel(), generator=gen, device=dev) < 0.5
        i, j = torch.where(swap, j, i), torch.where(swap, i, j)
    return n, i.contiguous(), j.contiguous(), c.to(torch.float32).contiguous()


# ---------------------------------------------------------------------------------------------------------------
# preparation and one pass
# ---------------------------------------------------------------------------------------------------------------
def prepare(case, seed):
    n, i, j, c = _instance(case, seed)
    state = dict(case=case, rama=Rama("cuda:0"), n=n, i=i, j=j, c=c, room=_room(case))
    if case["op"] == "static":      # the caller of the allocation-free entry point brings the labels array
        state["labels"] = torch.empty(n, dtype=torch.int32, device="cuda:0")
    if case["op"] == "mp":          # the cycles are what an earlier separation found
        state["cycles"] = state["rama"].find_conflicted_cycles(n, i, j, c, max_cycle_len=5)
    if case["op"] == "dual":
        state["params"] = default_params(dual_rounds=case["rounds"])
    torch.cuda.synchronize()
    return state


def run(state):
    case, rama = state["case"], state["rama"]
    graph = (state["n"], state["i"], state["j"], state["c"])
    op = case["op"]
    if op in ("solve", "static"):
        r = rama.solve(*graph, static=op == "static", labels=state.get("labels"))
        return [r["labels"], r["primal"], r["lower_bound"], r["rounds"], r["n_clusters"]]
    room = state["room"]
    if op == "cycles":
        lists = rama.find_conflicted_cycles(*graph, max_cycle_len=case["length"])
        return [_keep(state, str(q), x, room[q]) for q, x in enumerate(lists)] + [x.shape[0] for x in lists]
    if op == "mp":
        r = rama.message_passing(*graph, state["cycles"], case["k"])
    elif op == "contract":
        r = rama.contract(*graph, repeat=case["repeat"])
    else:
        r = rama.dual_rounds(*graph, state["params"])
    out = [_keep(state, name, r[name], room) for name in ("i", "j", "c")] + [r["i"].numel()]
    if op == "mp":
        return out + [r["lower_bound"]]
    if op == "contract":
        return out + [r["mapping"], _keep(state, "diag", r["diag"], state["n"]), r["n_nodes"]]
    return out + [r["lower_bound"], r["n_triangles"]] + r["lb_trace"]


def _sizes(case):
    """Nodes and edges of the instance (for neighbour graphs to about one percent)."""
    if case["graph"] == "knn":
        n = case["n"]
        m = 3.53 * n
    else:
        shape, offsets = _shape_offsets(case)
        n = math.prod(shape)
        m = sum(math.prod(max(0, s - abs(k)) for k, s in zip(off, shape)) for off in offsets)
    return n, m * (1.01 if case["shuffled"] else 1.0)


# 3-, 4- and 5-cycles with one repulsive edge per node (measured)
CYCLES = {"knn": (0.97, 3.3, 10.2), "longrange": (0.0, 5.2, 0.0), "window": (20.0, 0.0, 0.0), "grid3d": (0.0, 0.98, 0.0)}


def _room(case):
    """How many entries of each output a caller with buffers of a fixed size holds ready, by name."""
    n, m = _sizes(case)
    m = int(m) + 64 if case["graph"] != "knn" else int(3.7 * n) + 64
    if case["op"] == "cycles":
        return [int(1.5 * per * n) + 4096 for per in CYCLES[case["graph"]][: case["length"] - 2]]
    if case["op"] == "mp":
        return int(m + 1.2 * n) + 64
    if case["op"] == "dual":
        return 12 * m
    return m        # a contracted graph has no more edges than the graph


def _keep(state, name, value, room):
    """Copies a result, whose size depends on the data, into a buffer of the program's own: zero behind its end."""
    key = "out_" + name
    if key not in state:
        state[key] = torch.zeros((room,) + tuple(value.shape[1:]), dtype=value.dtype, device=value.device)
    state[key][: value.shape[0]].copy_(value)
    return state[key]


def work(case):
    """The edge list is read once and the results are written once; how many cycles, chords and contracted edges there
    are follows from the recipes (measured, per node)."""
    n, m = _sizes(case)
    op, read = case["op"], 12 * m
    if op in ("solve", "static"):
        return {"bytes": read + 4 * n, "flops": 0}
    if op == "cycles":
        found = sum((q + 3) * CYCLES[case["graph"]][q] for q in range(case["length"] - 2))
        return {"bytes": read + 4 * found * n, "flops": 0}
    if op == "mp":          # 0.98 four-cycles per voxel come in, about as many chords go out with the edges
        triangles = 2 * 0.98 * n
        return {"bytes": read + 16 * 0.98 * n + 12 * (m + 0.98 * n), "flops": 70 * triangles * case["k"]}
    if op == "contract":    # a matching leaves 60 % of a volume's edges; "P" leaves next to none
        return {"bytes": read + 4 * n + (12 * 0.6 * m + 4 * 0.6 * n if case["repeat"] else 0), "flops": 0}
    return {"bytes": read + 12 * (1.8 if case["rounds"] == 1 else 5.0) * m, "flops": 0}     # edges and chords


def tolerance(case):
    """Lists, mappings, labels and counts are whole numbers and stay the same.  fp32 sums are taken in a stated order
    (input position, ascending triangle), and every decision hangs on them, so other sums are not another correct
    result; what is free is the order of the fp64 sums behind a primal cost or a bound (1e-15 seen), and, where a
    result is compared with one in 64 bits, the rounding of the fp32 state."""
    if case["op"] in ("solve", "static", "dual"):
        return {"rel": 1e-12}
    if case["op"] == "mp":
        return {"rel": 5e-7}        # 1.1e-7 seen against 64 bits
    if case["op"] == "contract":
        return {"rel": 1e-7}        # 1.2e-8 to 3e-8 seen
    return "exact"


# ---------------------------------------------------------------------------------------------------------------
# the same in 64 bits, in plain torch
# ---------------------------------------------------------------------------------------------------------------
def _canonical(n, i, j, c):
    """Sorted keys lo * n + hi and summed costs of a list without loops."""
    lo, hi = torch.minimum(i, j).to(torch.int64), torch.maximum(i, j).to(torch.int64)
    key, inv = torch.unique(lo * n + hi, return_inverse=True)
    return key, torch.zeros(key.numel(), dtype=torch.float64, device=c.device).index_add_(0, inv, c.to(torch.float64))


def _square_cycles(shape, n, key, cost):
    """All 4-cycles of a 3-D grid (its unit squares) with exactly one repulsive edge, as fan triangles (a, b, c) and
    chords (p, q).  The square's corners are x, x+u, x+u+v, x+v; the grid is bipartite, so there are no others up to
    length 5."""
    ids = torch.arange(n, device=key.device).view(shape)
    tri, chord = [], []
    for u, v in ((0, 1), (0, 2), (1, 2)):
        def corner(a, b):
            sl = [slice(None)] * 3
            sl[u], sl[v] = slice(a, shape[u] - 1 + a), slice(b, shape[v] - 1 + b)
            return ids[tuple(sl)].reshape(-1)
        ring = [corner(0, 0), corner(1, 0), corner(1, 1), corner(0, 1)]
        c = torch.stack([cost[torch.searchsorted(key, torch.minimum(p, q) * n + torch.maximum(p, q))]
                         for p, q in zip(ring, ring[1:] + ring[:1])])
        one = ((c < 0).sum(0) == 1) & ((c > 0).sum(0) == 3)
        ring, at = torch.stack(ring)[:, one], (c < 0).to(torch.int64).argmax(0)[one]
        # the repulsive edge joins corners at and at + 1; the fan is drawn from the smaller of the two
        s = torch.arange(ring.shape[1], device=key.device)
        p, q = ring[at, s], ring[(at + 1) % 4, s]
        first = p < q
        v0 = torch.where(first, p, q)
        v1 = torch.where(first, ring[(at + 3) % 4, s], ring[(at + 2) % 4, s])
        v2 = torch.where(first, ring[(at + 2) % 4, s], ring[(at + 3) % 4, s])
        v3 = torch.where(first, q, p)
        tri += [torch.stack([v0, v1, v2]), torch.stack([v0, v2, v3])]
        chord.append(torch.minimum(v0, v2) * n + torch.maximum(v0, v2))
    return torch.cat(tri, 1).sort(0).values, torch.unique(torch.cat(chord))


def _message_passing(case, n, i, j, c, k):
    """Augmented edges, reduced costs and lower bound after k iterations, in fp64."""
    key, cost = _canonical(n, i, j, c)
    shape = (case["d"], case["h"], case["w"])
    tri, chord = _square_cycles(shape, n, key, cost)
    new = chord[~torch.isin(chord, key)]
    every, order = torch.cat([key, new]).sort()
    cost = torch.cat([cost, torch.zeros(new.numel(), dtype=torch.float64, device=key.device)])[order]
    e0 = torch.searchsorted(every, tri[0] * n + tri[1])
    e1 = torch.searchsorted(every, tri[0] * n + tri[2])
    e2 = torch.searchsorted(every, tri[1] * n + tri[2])
    known = torch.unique(e0 * every.numel() + e1, return_inverse=True)[1]      # a triangle is given by two of its edges
    first = torch.full((int(known.max()) + 1 if known.numel() else 0,), tri.shape[1], device=key.device)
    first.scatter_reduce_(0, known, torch.arange(tri.shape[1], device=key.device), "amin")
    edges = torch.stack([e0[first], e1[first], e2[first]])
    count = torch.bincount(edges.reshape(-1), minlength=every.numel())
    t = torch.zeros(edges.shape, dtype=torch.float64, device=key.device)

    def marginal(s):
        a, b, d = t[s], t[(s + 1) % 3], t[(s + 2) % 3]
        return torch.minimum(torch.minimum(a + b, a + d), a + b + d) - torch.clamp(b + d, max=0.0)

    for _ in range(k):
        t += (cost / count)[edges]
        out = torch.zeros_like(t)
        for s, weight in ((0, 1.0 / 3.0), (1, 0.5), (2, 1.0), (0, 0.5), (1, 1.0), (0, 1.0)):
            delta = weight * marginal(s)
            t[s] -= delta
            out[s] += delta
        sums = torch.zeros_like(cost).index_add_(0, edges.reshape(-1), out.reshape(-1))
        cost = torch.where(count > 0, sums, cost)
    a, b, d = t[0], t[1], t[2]
    worst = torch.stack([torch.zeros_like(a), a + b, a + d, b + d, a + b + d]).min(0).values
    return every, cost, float(torch.clamp(cost, max=0.0).sum() + worst.sum())


def _contract(n, i, j, c):
    """One handshake matching (larger cost first, then earlier edge) and the contracted graph; the matching takes its
    decisions on the costs as given in fp32, the sums are fp64."""
    key, cost = _canonical(n, i, j, c)
    u, v = key // n, key % n
    bits = cost.to(torch.float32).view(torch.int32).to(torch.int64)
    rank = (bits << 32) | (0xFFFFFFFF - torch.arange(key.numel(), device=key.device))
    mate = torch.full((n,), -1, dtype=torch.int64, device=key.device)
    left = cost > 0
    lu, lv, lr = u[left], v[left], rank[left]
    for _ in range(default_params().matching_rounds_cap):
        if lu.numel() == 0:
            break
        best = torch.zeros(n, dtype=torch.int64, device=key.device)
        best.scatter_reduce_(0, lu, lr, "amax")
        best.scatter_reduce_(0, lv, lr, "amax")
        hit = (best[lu] == lr) & (best[lv] == lr)
        mate[lu[hit]], mate[lv[hit]] = lv[hit], lu[hit]
        free = (mate[lu] < 0) & (mate[lv] < 0)
        lu, lv, lr = lu[free], lv[free], lr[free]
    node = torch.arange(n, device=key.device)
    rep = torch.where((mate >= 0) & (mate < node), mate, node)
    mapping = (torch.cumsum((rep == node).to(torch.int64), 0) - 1)[rep]
    n_new = int(mapping.max()) + 1
    a, b = mapping[u], mapping[v]
    diag = torch.zeros(n_new, dtype=torch.float64, device=key.device).index_add_(0, a[a == b], cost[a == b])
    new_key, new_cost = _canonical(n_new, a[a != b], b[a != b], cost[a != b])
    return mapping, new_key, new_cost, diag, n_new


def exact(case, seed):
    """Whole-number results and everything that hangs on a chain of fp32 decisions (labels, later rounds) have no
    64-bit value; the bound of a volume, one message-passing block and one contraction do."""
    op = case["op"]
    one_contraction = op == "contract" and case["repeat"] == 1 and not case["shuffled"]
    bound = op == "mp" or (op == "solve" and case["graph"] == "grid3d")
    if not (one_contraction or bound):
        return None
    n, i, j, c = _instance(case, seed)

    def padded(x, room):
        return torch.cat([x, torch.zeros(room - x.numel(), dtype=x.dtype, device=x.device)])

    if one_contraction:
        mapping, key, cost, diag, n_new = _contract(n, i, j, c)
        edges = [padded(x, _room(case)) for x in (key // n_new, key % n_new, cost)]
        return edges + [key.numel(), mapping, padded(diag, n), n_new]
    k = case["k"] if op == "mp" else default_params().mp_iters_first
    key, cost, lower = _message_passing(case, n, i, j, c, k)
    if op == "solve":
        return [None, None, lower, None, None]
    return [padded(x, _room(case)) for x in (key // n, key % n, cost)] + [key.numel(), lower]
