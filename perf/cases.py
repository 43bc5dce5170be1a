"""The measured workloads: one pass each through the library's public entry points.

Graphs are the families of this repository's configurations, tests and benchmark (2D and 3D grids,
RMAT, Erdos-Renyi, random geometric), symmetric int32 CSR without loops or duplicates and with sorted
rows, made on the GPU from the seed.  Shifts are Exp(beta) draws in units of 2^-20.
"""
import math

import numpy as np
import torch

import paper_1307_3692_amd as ldd

FIX = 20


# ------------------------------------------------------------------------------------------
# the cases
# ------------------------------------------------------------------------------------------
def listed():
    return [
        # one small mesh per call, where latency is everything (the 64 x 64 grid of the benchmark)
        dict(name="grid2d-64", op="decompose", graph="grid2d", x=64, y=64, beta=0.1),
        # the paper's experiment: a 1000 x 1000 grid, many rounds with small frontiers
        dict(name="grid2d-1000", op="decompose", graph="grid2d", x=1000, y=1000, beta=0.01),
        # a large mesh: hundreds of rounds (the benchmark's 256^3 grid)
        dict(name="grid3d-256", op="decompose", graph="grid3d", x=256, y=256, z=256, beta=0.02),
        # skewed graphs of few rounds: the smallest of the serving mix, a middle one, a large one
        # and the headline benchmark's scale 24
        dict(name="rmat-12", op="decompose", graph="rmat", scale=12, ef=16, beta=0.1),
        dict(name="rmat-16", op="decompose", graph="rmat", scale=16, ef=16, beta=0.05),
        dict(name="rmat-20", op="decompose", graph="rmat", scale=20, ef=16, beta=0.05),
        dict(name="rmat-24", op="decompose", graph="rmat", scale=24, ef=16, beta=0.05),
        # many uneven graphs in one call: the benchmark's 512, and a small batch of small graphs
        dict(name="batch-512", op="batch", graphs=512, n_lo=1000, n_hi=200000, b_lo=0.02, b_hi=0.3),
        dict(name="batch-48", op="batch", graphs=48, n_lo=700, n_hi=20000, b_lo=0.02, b_hi=0.3),
        # a burst of requests through the serving engine (scales and betas of the serving mix)
        dict(name="serve-64", op="serve", requests=64, s_lo=12, s_hi=22),
        # the Las Vegas loop: device-drawn shifts, decomposition, check of cut and radius
        dict(name="verified-rgg-150001", op="verified", graph="rgg", n=150001, deg=6.0, beta=0.05),
        # the block decomposition: one decomposition per level on the edges left
        dict(name="blocks-grid3d-64", op="blocks", graph="grid3d", x=64, y=64, z=64, beta=0.5),
    ]


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _draw_graph(rng, n_max):
    kind = rng.choice(("grid2d", "grid3d", "rmat", "er", "rgg"))
    if kind == "grid2d":
        n = _log_uniform(rng, 64, min(n_max, 4_000_000))
        x = max(2, round(math.sqrt(n) * rng.uniform(0.5, 2.0)))
        return dict(graph=kind, x=x, y=max(2, int(n / x)))
    if kind == "grid3d":
        n = _log_uniform(rng, 512, n_max)
        x = min(256, max(2, round(n ** (1 / 3) * rng.uniform(0.7, 1.4))))
        y = min(256, max(2, round(math.sqrt(n / x) * rng.uniform(0.7, 1.4))))
        return dict(graph=kind, x=x, y=y, z=min(256, max(2, int(n / x / y))))
    if kind == "rmat":
        return dict(graph=kind, scale=rng.randint(10, int(math.log2(n_max))), ef=rng.randint(4, 16))
    n = round(_log_uniform(rng, 1000, min(n_max, 2_000_000)))
    return dict(graph=kind, n=n, deg=round(rng.uniform(3.0, 10.0) if kind == "er" else rng.uniform(4.0, 8.0), 2))


def draw(rng):
    op = rng.choice(("decompose", "decompose", "decompose", "decompose", "batch", "batch", "serve", "verified",
                     "blocks"))
    if op == "batch":
        n_hi = round(_log_uniform(rng, 2000, 200_000))
        return dict(op=op, graphs=round(_log_uniform(rng, 8, 512)), n_lo=rng.randint(300, 1000), n_hi=n_hi, b_lo=0.02,
                    b_hi=0.3)
    if op == "serve":
        s_lo = rng.randint(10, 14)
        return dict(op=op, requests=round(_log_uniform(rng, 8, 64)), s_lo=s_lo, s_hi=rng.randint(s_lo, 22))
    n_max = {"decompose": 1 << 24, "verified": 1 << 20, "blocks": 1 << 18}[op]
    case = dict(op=op, **_draw_graph(rng, n_max))
    if op == "blocks":
        case["beta"] = round(rng.uniform(0.2, 0.5), 3)
    else:
        case["beta"] = round(_log_uniform(rng, 0.02, 0.3), 4)
    return case


# ------------------------------------------------------------------------------------------
# inputs
# ------------------------------------------------------------------------------------------
class _Draws:
    """Seeded draws on the GPU."""

    def __init__(self, seed):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(seed)

    def uniform(self, n, dtype=torch.float64):
        return torch.rand(n, generator=self.g, device="cuda", dtype=dtype)

    def randint(self, hi, n):
        return torch.randint(0, hi, (n,), generator=self.g, device="cuda")

    def shifts(self, n, beta):
        """floor(Exp(beta) * 2^20); beta a number or one per vertex."""
        return torch.floor(-torch.log1p(-self.uniform(n)) / beta * (1 << FIX)).to(torch.int64)


def _csr(n, src, dst, loops=True):
    """CSR of the undirected edges (both arcs, duplicates and loops dropped), ids below n."""
    if loops:
        keep = src != dst
        src, dst = src[keep], dst[keep]
    key = torch.cat((src * n + dst, dst * n + src))
    del src, dst
    key = torch.unique_consecutive(torch.sort(key)[0])
    row_ptr = torch.searchsorted(key, torch.arange(n + 1, device="cuda") * n).to(torch.int32)
    return row_ptr, (key % n).to(torch.int32)


def _grid(dims):
    ids = torch.arange(math.prod(dims), device="cuda").view(*dims)
    src, dst = [], []
    for k, d in enumerate(dims):
        src.append(ids.narrow(k, 0, d - 1).reshape(-1))
        dst.append(ids.narrow(k, 1, d - 1).reshape(-1))
    return _csr(ids.numel(), torch.cat(src), torch.cat(dst), loops=False)


def _rmat(d, scale, ef):
    """ef 2^scale Kronecker draws (a, b, c, d = .57, .19, .19, .05), relabelled at random."""
    n, m = 1 << scale, ef << scale
    src = torch.zeros(m, dtype=torch.int32, device="cuda")
    dst = torch.zeros(m, dtype=torch.int32, device="cuda")
    for _ in range(scale):
        u = d.uniform(m, torch.float32)
        src = 2 * src + (u >= 0.76)
        dst = 2 * dst + (((u >= 0.57) & (u < 0.76)) | (u >= 0.95))
        src, dst = src.to(torch.int32), dst.to(torch.int32)
    perm = torch.randperm(n, generator=d.g, device="cuda")
    return _csr(n, perm[src], perm[dst])


def _er_edges(d, sizes, deg, first):
    """Uniform pairs inside each graph (about deg n / 2 of them); graph i's ids start at first[i]."""
    m = (sizes.double() * deg / 2).round().long()
    g = torch.repeat_interleave(torch.arange(sizes.numel(), device="cuda"), m)
    n = sizes[g].double()
    total = g.numel()
    src = (d.uniform(total) * n).long() + first[g]
    return src, (d.uniform(total) * n).long() + first[g]


def _rgg_edges(d, sizes, deg, first):
    """Pairs of uniform points of each graph's unit square within r = sqrt(deg / (pi n))."""
    r = torch.sqrt(deg / (math.pi * sizes.double()))
    cells = torch.clamp(torch.floor(1 / r).long(), min=1)
    base = torch.cumsum(cells * cells, 0) - cells * cells
    g = torch.repeat_interleave(torch.arange(sizes.numel(), device="cuda"), sizes)
    pos = torch.arange(g.numel(), device="cuda") - torch.repeat_interleave(torch.cumsum(sizes, 0) - sizes, sizes)
    x, y = d.uniform(g.numel()), d.uniform(g.numel())
    k = cells[g]
    cx, cy = torch.minimum((x * k).long(), k - 1), torch.minimum((y * k).long(), k - 1)
    cell, order = torch.sort(base[g] + cx * k + cy)
    start = torch.searchsorted(cell, torch.arange(int((cells * cells).sum()) + 1, device="cuda"))
    x, y, cx, cy, g, k, v = x[order], y[order], cx[order], cy[order], g[order], k[order], pos[order]
    v = v + first[g]
    me = torch.arange(g.numel(), device="cuda")
    src, dst = [], []
    for dx in (0, 1):  # a pair is found from its end in the lower strip (in one strip: the earlier point)
        ok = cx + dx < k
        row = base[g] + torch.where(ok, cx + dx, cx) * k
        lo = start[row + torch.clamp(cy - 1, min=0)]
        hi = start[row + torch.minimum(cy + 1, k - 1) + 1]
        if dx == 0:
            lo = torch.maximum(lo, me + 1)
        cnt = torch.where(ok, torch.clamp(hi - lo, min=0), 0)
        a = torch.repeat_interleave(me, cnt)
        b = torch.arange(a.numel(), device="cuda") + (lo - (torch.cumsum(cnt, 0) - cnt))[a]
        near = (x[a] - x[b]) ** 2 + (y[a] - y[b]) ** 2 <= (r * r)[g[a]]
        src.append(v[a[near]])
        dst.append(v[b[near]])
    return torch.cat(src), torch.cat(dst)


def _graph(d, case):
    if case["graph"] == "grid2d":
        return _grid((case["x"], case["y"]))
    if case["graph"] == "grid3d":
        return _grid((case["x"], case["y"], case["z"]))
    if case["graph"] == "rmat":
        return _rmat(d, case["scale"], case["ef"])
    sizes, first = torch.tensor([case["n"]], device="cuda"), torch.zeros(1, dtype=torch.long, device="cuda")
    edges = _er_edges if case["graph"] == "er" else _rgg_edges
    return _csr(case["n"], *edges(d, sizes, case["deg"], first))


def _batch_sizes(case):
    """Vertices of the batch's graphs: log-uniform, the same for every seed (even ones are
    Erdos-Renyi of mean degree 8, odd ones random geometric of mean degree 6)."""
    u = (np.arange(case["graphs"]) * 0.6180339887498949) % 1.0
    return np.floor(case["n_lo"] * (case["n_hi"] / case["n_lo"]) ** u).astype(np.int64)


def _batch(d, case):
    """(vtx_off, arc_off) on the host, and row_ptr, col_idx (local ids), shift_fix packed on the GPU."""
    sizes = _batch_sizes(case)
    G = sizes.size
    vo = np.concatenate(([0], np.cumsum(sizes)))
    ds, first = torch.from_numpy(sizes).cuda(), torch.from_numpy(vo[:-1].copy()).cuda()
    even = torch.arange(0, G, 2, device="cuda")
    odd = torch.arange(1, G, 2, device="cuda")
    se, de = _er_edges(d, ds[even], 8.0, first[even])
    so, do = _rgg_edges(d, ds[odd], 6.0, first[odd]) if G > 1 else (se[:0], de[:0])
    n = int(vo[-1])
    rp, ci = _csr(n, torch.cat((se, so)), torch.cat((de, do)))
    gid = torch.repeat_interleave(torch.arange(G, device="cuda"), ds)
    ao = rp[torch.from_numpy(vo).cuda()].long()
    # local row offsets, G + n of them: vertex v of graph g at v + g, and each graph's end
    rows = torch.empty(n + G, dtype=torch.int32, device="cuda")
    v = torch.arange(n, device="cuda")
    rows[v + gid] = (rp[:-1].long() - ao[gid]).to(torch.int32)
    g = torch.arange(G, device="cuda")
    rows[torch.from_numpy(vo[1:].copy()).cuda() + g] = (ao[1:] - ao[:-1]).to(torch.int32)
    row = torch.repeat_interleave(v, (rp[1:] - rp[:-1]).long())
    local = (ci - first[gid[row]].to(torch.int32)).contiguous()
    beta = torch.exp(d.uniform(G) * math.log(case["b_hi"] / case["b_lo"])) * case["b_lo"]
    return vo, ao.cpu().numpy(), rows, local, d.shifts(n, beta[gid])


def _requests(d, case):
    """One RMAT graph per scale; request i takes the next scale and beta, with shifts of its own."""
    graphs = {s: _rmat(d, s, 16) for s in range(case["s_lo"], case["s_hi"] + 1)}
    out = []
    for i in range(case["requests"]):
        rp, ci = graphs[case["s_lo"] + (7 * i) % len(graphs)]
        out.append((rp, ci, d.shifts(rp.numel() - 1, (0.05, 0.1, 0.2)[i % 3])))
    return out


def prepare(case, seed):
    d = _Draws(seed)
    st = dict(case=case, seed=seed)
    if case["op"] == "batch":
        st["args"] = _batch(d, case)
    elif case["op"] == "serve":
        st["requests"] = _requests(d, case)
        off = np.concatenate(([0], np.cumsum([s.numel() for _, _, s in st["requests"]])))
        st["centre"] = torch.empty(int(off[-1]), dtype=torch.int32, device="cuda")
        st["parts"] = [st["centre"][a:b] for a, b in zip(off[:-1], off[1:])]
        st["server"] = ldd.Server(hbm_budget_bytes=4 << 30)
    else:
        # (a level per arc comes back from the block decomposition: one graph for every seed of its draws)
        st["rp"], st["ci"] = _graph(_Draws(1) if case["op"] == "blocks" else d, case)
        if case["op"] == "decompose":
            st["s"] = d.shifts(st["rp"].numel() - 1, case["beta"])
    return st


# ------------------------------------------------------------------------------------------
# one pass
# ------------------------------------------------------------------------------------------
def run(st):
    case = st["case"]
    if case["op"] == "decompose":
        centre, cut = ldd.decompose(st["rp"], st["ci"], st["s"], case["beta"])
        return dict(centre=centre, cut=cut)
    if case["op"] == "batch":
        centre, cuts = ldd.decompose_batch(*st["args"])
        return dict(centre=centre, cut=np.array(cuts))
    if case["op"] == "serve":
        srv = st["server"]
        tickets = [srv.submit(*q, centre=c) for q, c in zip(st["requests"], st["parts"])]
        return dict(centre=st["centre"], cut=np.array([srv.wait(t)[1] for t in tickets]))
    if case["op"] == "verified":
        centre, shifts, rep = ldd.decompose_verified(st["rp"], st["ci"], case["beta"], st["seed"])
        return dict(centre=centre, shifts=shifts, cut=rep["cut_edges"], radius=rep["max_radius"],
                    attempts=rep["attempts"])
    level, edges = ldd.block_decompose(st["rp"], st["ci"], beta=case["beta"], seed=st["seed"])
    return dict(level=level, edges=np.array(edges + [0] * (64 - len(edges))))  # 64 levels at most


# ------------------------------------------------------------------------------------------
# what a pass cannot do without
# ------------------------------------------------------------------------------------------
def _rmat_arcs(scale, ef):
    """Expected arcs of _rmat: a cell with i a's, j of b or c, k d's has probability a^i b^j d^k, and
    an edge is missing when none of the draws hits its two cells."""
    draws, arcs = ef << scale, 0.0
    for j in range(1, scale + 1):  # j = 0 is the diagonal: loops
        for k in range(scale - j + 1):
            p = 2 * 0.57 ** (scale - j - k) * 0.19 ** j * 0.05 ** k
            cells = math.comb(scale, j) * math.comb(scale - j, k) * 2.0 ** j
            arcs += cells * -math.expm1(draws * math.log1p(-p))
    return arcs


def _er_arcs(n, deg):
    return deg * n


def _rgg_arcs(n, deg):
    r = math.sqrt(deg / (math.pi * n))
    return n * (n - 1) * min(1.0, math.pi * r ** 2 - 8 / 3 * r ** 3 + r ** 4 / 2)  # the square's border counted


def _sizes(case):
    """(vertices, arcs) of a case's graph."""
    if case["graph"] in ("grid2d", "grid3d"):
        dims = [case[k] for k in "xyz" if k in case]
        n = math.prod(dims)
        return n, 2 * sum(n // d * (d - 1) for d in dims)
    if case["graph"] == "rmat":
        return 1 << case["scale"], _rmat_arcs(case["scale"], case["ef"])
    return case["n"], (_er_arcs if case["graph"] == "er" else _rgg_arcs)(case["n"], case["deg"])


def work(case):
    """CSR (4 B per row and arc) and shifts (8 B) read, centres (4 B) written; one comparison per arc."""
    if case["op"] == "batch":
        sizes = _batch_sizes(case)
        n = int(sizes.sum())
        nnz = sum((_rgg_arcs(int(k), 6.0) if i % 2 else _er_arcs(int(k), 8.0)) for i, k in enumerate(sizes))
    elif case["op"] == "serve":
        scales = [case["s_lo"] + (7 * i) % (case["s_hi"] - case["s_lo"] + 1) for i in range(case["requests"])]
        n = sum(1 << s for s in scales)
        nnz = sum(_rmat_arcs(s, 16) for s in scales)
    else:
        n, nnz = _sizes(case)
        if case["op"] == "blocks":  # the graph read, a level per arc written
            return dict(bytes=int(4 * n + 8 * nnz), flops=int(nnz))
    # (the Las Vegas loop writes its shifts where the others read theirs)
    return dict(bytes=int(16 * n + 4 * nnz), flops=int(nnz))


# ------------------------------------------------------------------------------------------
# the same results, plainly
# ------------------------------------------------------------------------------------------
def _reference(rp, ci, s):
    """centre(v) = the u with the least (2^20 dist(u, v) - shift(u), u), by relaxing every arc of a
    changed vertex until no label drops; and which arcs are cut."""
    n = rp.numel() - 1
    bits = max(1, (n - 1).bit_length())
    row = torch.repeat_interleave(torch.arange(n, device="cuda"), (rp[1:] - rp[:-1]).long())
    label = ((s.max() - s) << bits) | torch.arange(n, device="cuda")
    changed = torch.ones(n, dtype=torch.bool, device="cuda")
    while bool(changed.any()):
        arc = torch.nonzero(changed[row]).squeeze(1)
        to, offer = ci[arc].long(), label[row[arc]] + (1 << (FIX + bits))
        better = offer < label[to]
        new = label.scatter_reduce(0, to[better], offer[better], "amin")
        changed, label = new < label, new
    centre = (label & ((1 << bits) - 1)).to(torch.int32)
    return centre, centre[row] != centre[ci.long()]


def exact(case, seed):
    if case["op"] in ("verified", "blocks"):  # their shifts are drawn by the library
        return None
    st = prepare(case, seed)
    if case["op"] == "decompose":
        centre, is_cut = _reference(st["rp"], st["ci"], st["s"])
        return dict(centre=centre, cut=int(is_cut.sum()) // 2)
    if case["op"] == "batch":  # the disjoint union: ids keep their order inside every graph
        vo, ao, rows, local, s = st["args"]
        G, n = len(vo) - 1, int(vo[-1])
        first, arcs = torch.from_numpy(vo[:-1].copy()).cuda(), torch.from_numpy(ao.copy()).cuda()
        gid = torch.repeat_interleave(torch.arange(G, device="cuda"), torch.from_numpy(np.diff(vo)).cuda())
        rp = torch.cat((rows[torch.arange(n, device="cuda") + gid] + arcs[gid], arcs[-1:]))
        of_arc = torch.repeat_interleave(torch.arange(G, device="cuda"), arcs[1:] - arcs[:-1])
        centre, is_cut = _reference(rp, local + first[of_arc], s)
        cut = torch.bincount(of_arc[is_cut], minlength=G) // 2
        return dict(centre=(centre - first[gid]).to(torch.int32), cut=cut.cpu().numpy())
    st["server"].close()
    parts = [_reference(*q) for q in st["requests"]]
    return dict(centre=torch.cat([p[0] for p in parts]), cut=np.array([int(p[1].sum()) // 2 for p in parts]))
