"""Workloads of the connected-components library, as a user's program calls it.

Every case is one public call (or, for the request server, one burst of
requests) on inputs resident where that call takes them.  The graph families
are the library's own: uniform random pairs with a few isolated 4-cliques,
R-MAT (.57/.19/.19/.05, ids relabelled by a random permutation), 4-neighbour
lattices with 30 % of the edges deleted, batches of independent uniform graphs
with log-uniform sizes and degrees, and a stream of R-MAT requests.  Inputs
are drawn on the GPU from the seed alone; sizes depend on the case alone.

  listed()             the named cases
  draw(rng)            one more case of the same ranges
  prepare(case, seed)  inputs in hand before the call
  run(state)           the call; returns every label it computed
  work(case)           bytes one call cannot do without (inputs read once,
                       labels written once)
"""
import math

import numpy as np
import torch

import paper_1612_01178_amd as cc

DEV = "cuda"
RMAT_A, RMAT_B, RMAT_C = 0.57, 0.19, 0.19
MAX_ENTRIES = 1 << 29  # of one pair list
SERVER_BYTES = 16 << 30


def listed():
    return [
        # a query on a small graph (a neighbourhood, a molecule set): launch
        # and call latency, nothing else
        dict(name="er_small", op="labels", family="er", n=1000, m=4000),
        # a mid-size uniform random graph, all of it in cache
        dict(name="er_64k", op="labels", family="er", n=65536, m=524672),
        # a social graph of the request stream's middle, each edge listed once,
        # with an odd entry count
        dict(name="rmat_18", op="labels", family="rmat", scale=18, m=2621441, symmetrize=False),
        # a social graph near the top of the request stream
        dict(name="rmat_21", op="labels", family="rmat", scale=21, m=24 << 21, symmetrize=False),
        # the largest: a social graph of 2^24 vertices, both orientations listed
        dict(name="rmat_24_sym", op="labels", family="rmat", scale=24, m=16 << 24, symmetrize=True),
        # a city's road map or a segmentation mask: a lattice with odd sides
        dict(name="grid_odd", op="labels", family="grid", width=1237, height=1001),
        # a continent's road map
        dict(name="grid_4096", op="labels", family="grid", width=4096, height=4096),
        # a social graph that the program already holds as an adjacency
        dict(name="csr_rmat_20", op="csr", family="rmat", scale=20, m=16 << 20, symmetrize=True),
        # a road map as an adjacency
        dict(name="csr_grid_2k", op="csr", family="grid", width=2048, height=2048, symmetrize=True),
        # many molecule-sized graphs per call, their offsets on the host
        dict(name="batch_tiny", op="batch", count=2000, lo_exp=4.0, hi_exp=8.0, deg_hi=8.0,
             shape_seed=1),
        # 10,000 graphs of 256 to 65,536 vertices, offsets on the device
        dict(name="batch_10k", op="batch_device", count=10000, lo_exp=8.0, hi_exp=16.0,
             deg_hi=16.0, shape_seed=1004),
        # a burst of requests to the server: R-MAT graphs of scale 10 to 22
        dict(name="serve_burst", op="serve", count=24, scale_lo=10, scale_hi=22, ef_lo=8,
             ef_hi=32, shape_seed=1005),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["er", "er", "rmat", "rmat", "grid", "grid", "csr_rmat", "csr_grid", "batch",
                       "batch_device", "serve"])
    if kind == "er":
        n = _log_uniform(rng, 300, 4 << 20)
        m = max(1, min(1 << 25, int(n * math.exp(rng.uniform(math.log(0.5), math.log(32))))))
        return dict(op="labels", family="er", n=n, m=m)
    if kind in ("rmat", "csr_rmat"):
        scale = rng.randint(12, 23) if kind == "rmat" else rng.randint(12, 21)
        sym = kind == "csr_rmat" or rng.random() < 0.3
        # an entry factor that is no whole number, so the list has a ragged end
        m = int((1 << scale) * math.exp(rng.uniform(math.log(6), math.log(32 if not sym else 16))))
        m = min(m, MAX_ENTRIES // 2)
        op = "labels" if kind == "rmat" else "csr"
        return dict(op=op, family="rmat", scale=scale, m=m, symmetrize=sym)
    if kind in ("grid", "csr_grid"):
        width = _log_uniform(rng, 40, 4096)
        height = _log_uniform(rng, 40, 4096)
        case = dict(op="labels" if kind == "grid" else "csr", family="grid", width=width,
                    height=height)
        if kind == "csr_grid":
            case["symmetrize"] = True
        return case
    if kind == "serve":
        return dict(op="serve", count=rng.randint(8, 32), scale_lo=10, scale_hi=rng.randint(14, 22),
                    ef_lo=8, ef_hi=32, shape_seed=rng.randrange(1 << 30))
    lo = rng.uniform(4.0, 10.0)
    hi = min(16.0, lo + rng.uniform(1.0, 6.0))
    mean_n = 2 ** ((lo + hi) / 2)
    count = min(_log_uniform(rng, 20, 10000), max(20, int((1 << 27) / mean_n)))
    return dict(op=kind, count=count, lo_exp=round(lo, 2), hi_exp=round(hi, 2),
                deg_hi=round(rng.uniform(4.0, 16.0), 1), shape_seed=rng.randrange(1 << 30))


# ------------------------------------------------------------------ sizes
def _grid_entries(case):
    w, h = case["width"], case["height"]
    edges = w * (h - 1) + h * (w - 1)
    return edges - edges * 3 // 10


def _pair_sizes(case):
    """(n, entries) of a single graph."""
    if case["family"] == "er":
        return case["n"], case["m"]
    if case["family"] == "rmat":
        return 1 << case["scale"], case["m"] * (2 if case["symmetrize"] else 1)
    m = _grid_entries(case)
    return case["width"] * case["height"], m * (2 if case.get("symmetrize") else 1)


def _batch_sizes(case):
    """Vertex and entry counts of a batch's graphs: both log-uniform."""
    r = np.random.RandomState(case["shape_seed"] % (1 << 32))
    c = case["count"]
    nv = np.rint(2.0 ** r.uniform(case["lo_exp"], case["hi_exp"], c)).astype(np.int64)
    deg = case["deg_hi"] ** r.uniform(0.0, 1.0, c)
    return nv, np.rint(deg * nv / 2.0).astype(np.int64)


def _serve_sizes(case):
    r = np.random.RandomState(case["shape_seed"] % (1 << 32))
    c = case["count"]
    scales = r.randint(case["scale_lo"], case["scale_hi"] + 1, c)
    efs = r.randint(case["ef_lo"], case["ef_hi"] + 1, c)
    return [(int(s), int(e) << int(s)) for s, e in zip(scales, efs)]


def work(case):
    if case["op"] in ("labels", "csr"):
        n, m = _pair_sizes(case)
        nbytes = 8 * m + 4 * n if case["op"] == "labels" else 4 * m + 8 * (n + 1) + 4 * n
    elif case["op"] == "serve":
        nbytes = sum(8 * m + (4 << s) for s, m in _serve_sizes(case))
    else:
        nv, me = _batch_sizes(case)
        nbytes = 8 * int(me.sum()) + 4 * int(nv.sum()) + 16 * (len(nv) + 1)
    return {"bytes": nbytes, "flops": 0}


# ------------------------------------------------------------------ inputs
def _uniform(gen, n, m):
    """m entries: the six edges of each of n / 1024 isolated 4-cliques (at
    least one), and before them uniform pairs over the other vertices."""
    cliques = min(max(1, n // 1024), m // 6)
    perm = torch.randperm(n, generator=gen, device=DEV, dtype=torch.int32)
    members, pool = perm[: 4 * cliques].view(cliques, 4), perm[4 * cliques:]
    ends = []
    for side in ([0, 0, 0, 1, 1, 2], [1, 2, 3, 2, 3, 3]):
        i = torch.randint(0, pool.numel(), (m - 6 * cliques,), generator=gen, device=DEV)
        ends.append(torch.cat([pool[i], members[:, side].reshape(-1)]))
    return ends


def _rmat(gen, scale, m, symmetrize):
    n = 1 << scale
    total = 2 * m if symmetrize else m
    u = torch.empty(total, dtype=torch.int32, device=DEV)
    v = torch.empty(total, dtype=torch.int32, device=DEV)
    perm = torch.randperm(n, generator=gen, device=DEV, dtype=torch.int32)
    chunk = 1 << 25
    for e0 in range(0, m, chunk):
        k = min(chunk, m - e0)
        x = torch.zeros(k, dtype=torch.int32, device=DEV)
        y = torch.zeros(k, dtype=torch.int32, device=DEV)
        for _ in range(scale):
            r = torch.rand(k, generator=gen, device=DEV)
            lower = r >= RMAT_A + RMAT_B
            right = torch.where(lower, r >= RMAT_A + RMAT_B + RMAT_C, r >= RMAT_A)
            x.mul_(2).add_(lower)
            y.mul_(2).add_(right)
        u[e0:e0 + k] = perm[x]
        v[e0:e0 + k] = perm[y]
    if symmetrize:
        u[m:] = v[:m]
        v[m:] = u[:m]
    return u, v


def _grid(gen, w, h):
    """Row-major lattice: each vertex's right, then down neighbour, in id
    order, with 30 % of the edges deleted."""
    ids = torch.arange(w * h, dtype=torch.int32, device=DEV).view(h, w)
    a = ids.unsqueeze(2).expand(h, w, 2).reshape(-1)
    b = torch.stack([ids + 1, ids + w], 2).reshape(-1)
    ok = torch.ones(h, w, 2, dtype=torch.bool, device=DEV)
    ok[:, w - 1, 0] = False
    ok[h - 1, :, 1] = False
    ok = ok.reshape(-1)
    a, b = a[ok], b[ok]
    edges = a.numel()
    gone = torch.randperm(edges, generator=gen, device=DEV)[: edges * 3 // 10]
    keep = torch.ones(edges, dtype=torch.bool, device=DEV)
    keep[gone] = False
    return a[keep].contiguous(), b[keep].contiguous()


def _pairs(case, gen):
    n, _ = _pair_sizes(case)
    if case["family"] == "er":
        return (n, *_uniform(gen, n, case["m"]))
    if case["family"] == "rmat":
        u, v = _rmat(gen, case["scale"], case["m"], case["symmetrize"])
    else:
        u, v = _grid(gen, case["width"], case["height"])
        if case.get("symmetrize"):
            u, v = torch.cat([u, v]), torch.cat([v, u])
    return n, u, v


def _adjacency(n, u, v):
    """row_ptr and col of the pairs, columns ascending within a row."""
    key, _ = torch.sort(u.to(torch.int64) * n + v)
    row_ptr = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    torch.cumsum(torch.bincount(u, minlength=n), 0, out=row_ptr[1:])
    return row_ptr, (key % n).to(torch.int32)


def _batch(case, gen):
    nv, me = _batch_sizes(case)
    vo = np.concatenate([[0], np.cumsum(nv)]).astype(np.int64)
    eo = np.concatenate([[0], np.cumsum(me)]).astype(np.int64)
    top = torch.repeat_interleave(torch.from_numpy(nv).to(DEV), torch.from_numpy(me).to(DEV))
    ends = []
    for _ in range(2):
        r = torch.rand(top.numel(), generator=gen, device=DEV, dtype=torch.float64)
        ends.append(torch.minimum((r * top).to(torch.int64), top - 1).to(torch.int32))
    return vo, eo, ends[0], ends[1], int(nv.max())


_server = None


def _the_server():
    """The one server a serving program keeps for its life."""
    global _server
    if _server is None:
        _server = cc.Server(device_bytes=SERVER_BYTES, workers=3)
    return _server


def prepare(case, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(int(seed))
    op = case["op"]
    if op == "labels":
        n, u, v = _pairs(case, gen)
        return dict(op=op, n=n, u=u, v=v, out=torch.empty(n, dtype=torch.int32, device=DEV))
    if op == "csr":
        n, u, v = _pairs(case, gen)
        row_ptr, col = _adjacency(n, u, v)
        return dict(op=op, n=n, row_ptr=row_ptr, col=col,
                    out=torch.empty(n, dtype=torch.int32, device=DEV))
    if op == "serve":
        graphs = [(*_rmat(gen, s, m, False), 1 << s,
                   torch.empty(1 << s, dtype=torch.int32, device=DEV))
                  for s, m in _serve_sizes(case)]
        return dict(op=op, server=_the_server(), graphs=graphs)
    vo, eo, u, v, max_n = _batch(case, gen)
    out = torch.empty(int(vo[-1]), dtype=torch.int32, device=DEV)
    if op == "batch":
        return dict(op=op, u=u, v=v, vo=vo, eo=eo, out=out)
    return dict(op=op, u=u, v=v, vo=torch.from_numpy(vo).to(DEV), eo=torch.from_numpy(eo).to(DEV),
                max_n=max_n, out=out)


def run(state):
    s = state
    if s["op"] == "labels":
        return cc.labels(s["u"], s["v"], s["n"], out=s["out"])
    if s["op"] == "csr":
        return cc.labels_csr(s["row_ptr"], s["col"], s["n"], out=s["out"])
    if s["op"] == "batch":
        return cc.labels_batch(s["u"], s["v"], s["vo"], s["eo"], out=s["out"])
    if s["op"] == "batch_device":
        return cc.labels_batch_device(s["u"], s["v"], s["vo"], s["eo"], s["max_n"], s["out"])
    tickets = [s["server"].submit(u, v, n, out) for u, v, n, out in s["graphs"]]
    return [s["server"].wait(t)[0] for t in tickets]
