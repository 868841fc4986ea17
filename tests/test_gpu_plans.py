"""The automatic plan's paths at the sizes where its rules change and its
kernels have edges, against the CPU oracle (integer labels with one correct
answer: every comparison is bit-exact)."""
import time

import numpy as np
import pytest

import graphgen
import oracle

torch = pytest.importorskip("torch")
import paper_1612_01178_amd as cc  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    cc.load()
    return torch.device("cuda:0")


def put(x, dev, offset=0):
    """x on the device, its base `offset` words past a 16-byte boundary."""
    t = torch.zeros(len(x) + offset, dtype=torch.int32, device=dev)
    t[offset:] = torch.from_numpy(np.ascontiguousarray(x, dtype=np.int32)).to(dev)
    return t[offset:]


# (n, m): one vertex, no entries, a partial and a full step of 8,192 entries,
# one and two segments, the last sizes solved by one workgroup in LDS and the
# first ones past them
@pytest.mark.parametrize("n,m", [(1, 0), (1, 3), (5, 0), (64, 1), (100, 8191), (100, 8192),
                                 (100, 32769), (1025, 40000), (32768, 65536), (32768, 65537),
                                 (32769, 100), (16384, 98304), (16385, 98304), (300, 130472)])
def test_small_lists(dev, n, m):
    u, v = graphgen.uniform_pairs(m, n, seed=n + m, stream=0)
    want = oracle.labels(u, v, n)
    for offset in (0, 1):
        print("small", n, m, offset, flush=True)
        du, dv = put(u, dev, offset), put(v, dev, offset)
        lab, st = cc.labels(du, dv, n, return_stats=True)
        assert np.array_equal(lab.cpu().numpy(), want)
        assert st["host_syncs"] >= 1 and st["giant_label"] == -1
        out = torch.full((n,), -7, dtype=torch.int32, device=dev)
        cc.labels_noalloc(du, dv, n, out=out)
        assert np.array_equal(out.cpu().numpy(), want)
        for opt in (cc.Options(path_halving="off"), cc.Options(no_sync=True), cc.Options(graph=True),
                    cc.Options(profile=True)):
            out.fill_(-7)
            cc.labels(du, dv, n, out=out, options=opt)
            torch.cuda.synchronize()
            assert np.array_equal(out.cpu().numpy(), want), opt
        assert cc.stream_status() == cc.CC_OK
    if m:
        u[m // 2] = n
        for opt in (cc.Options(), cc.Options(no_sync=True)):
            with pytest.raises(cc.CCError) as ei:
                cc.labels(put(u, dev), put(v, dev), n, options=opt)
                torch.cuda.synchronize()
                cc.stream_status()
            assert ei.value.code == cc.CC_ERR_RANGE


# (count, lo, hi): vertex counts log-uniform in [lo, hi].  One graph, a launch
# without preparation at each workgroup size, the last and first counts on
# either side of its rule, more graphs than workgroups (every queue drawn
# from), the first sizes with 16-bit slots
@pytest.mark.parametrize("count,lo,hi", [(1, 1, 1), (7, 1, 3), (512, 200, 256), (513, 200, 256),
                                         (9000, 1, 40), (512, 300, 1024), (2049, 257, 1024),
                                         (300, 1025, 4096), (1100, 1025, 4096), (4100, 700, 1025),
                                         (600, 4097, 8192), (40, 30000, 32768), (40, 30000, 32769)])
def test_batches_by_rule(dev, count, lo, hi):
    rng = np.random.default_rng(count + hi)
    nv = np.exp(rng.uniform(np.log(lo), np.log(hi + 0.5), count)).astype(np.int64)
    nv[rng.integers(0, count)] = hi
    me = (nv * rng.uniform(0, 3, count)).astype(np.int64)
    if count > 5:
        nv[3] = me[3] = me[4] = 0
    vo = np.concatenate([[0], np.cumsum(nv)])
    eo = np.concatenate([[0], np.cumsum(me)])
    top = np.repeat(nv, me)
    u = (rng.random(len(top)) * top).astype(np.int32)
    v = (rng.random(len(top)) * top).astype(np.int32)
    want = oracle.labels_batch(u, v, vo, eo)
    du, dv = put(u, dev), put(v, dev)
    dvo, deo = torch.from_numpy(vo).to(dev), torch.from_numpy(eo).to(dev)
    side = torch.cuda.Stream()
    for opt in (cc.Options(), cc.Options(path_halving="off"), cc.Options(block=64, segments=3),
                cc.Options(graph=True)):
        print("batch", count, lo, hi, opt.block, opt.graph, flush=True)
        for rep in range(2 if opt.graph else 1):
            assert np.array_equal(cc.labels_batch(du, dv, vo, eo, options=opt,
                                                  stream=side).cpu().numpy(), want), opt
            out = torch.full((len(want),), -7, dtype=torch.int32, device=dev)
            torch.cuda.synchronize()
            cc.labels_batch_device(du, dv, dvo, deo, hi, out, options=opt, stream=side)
            assert np.array_equal(out.cpu().numpy(), want), opt
    if me[-1] > 0:
        u[-1] = nv[-1]
        du = put(u, dev)
        for call in (lambda: cc.labels_batch(du, dv, vo, eo),
                     lambda: cc.labels_batch_device(du, dv, dvo, deo, hi, out)):
            with pytest.raises(cc.CCError) as ei:
                call()
            assert ei.value.code == cc.CC_ERR_RANGE
    if hi > 1:
        with pytest.raises(cc.CCError) as ei:
            cc.labels_batch_device(put(v, dev), dv, dvo, deo, hi - 1, out)
        assert ei.value.code == cc.CC_ERR_ARG


# (scale, entries, both orientations): the filtered plan at the first list it
# takes, with rounds over a prefix and without, the bitmap in LDS at one and
# two workgroups per CU, a ragged end; the largest bitmap in LDS and the first
# size with the vertex table are below
@pytest.mark.parametrize("scale,m,sym", [(10, 1 << 21, False), (17, (1 << 21) + 5, False),
                                         (19, 1 << 21, True), (20, (1 << 23) + 3, False)])
def test_filtered_plan(dev, scale, m, sym):
    u, v, n = graphgen.rmat(scale, 0, seed=scale + m, m=m, symmetrize=sym)
    want = oracle.labels(u, v, n)
    for offset in (0, 3):
        du, dv = put(u, dev, offset), put(v, dev, offset)
        for opt in (cc.Options(), cc.Options(path_halving="off"), cc.Options(hook="atomic", filter="giant"),
                    cc.Options(hook="atomic", filter="giant", hot_cache="vertex"),
                    cc.Options(symmetric=True) if sym else cc.Options(no_sync=True)):
            print("filtered", scale, m, offset, opt, flush=True)
            out = torch.full((n,), -7, dtype=torch.int32, device=dev)
            cc.labels(du, dv, n, out=out, options=opt)
            torch.cuda.synchronize()
            assert np.array_equal(out.cpu().numpy(), want), opt
    for at in (0, m // 2, len(u) - 1):
        keep, u[at] = u[at], n
        with pytest.raises(cc.CCError) as ei:
            cc.labels(put(u, dev), dv, n)
        assert ei.value.code == cc.CC_ERR_RANGE
        u[at] = keep


@pytest.mark.parametrize("n", [160 * 1024 * 8 - 31, 160 * 1024 * 8, 160 * 1024 * 8 + 1,
                               320 * 1024 * 8, 320 * 1024 * 8 + 1])
def test_filtered_plan_at_the_lds_bitmap_limit(dev, n):
    """Half of the ids joined by a cycle and random chords, the rest in pairs
    or alone: a giant component whose bitmap ends in a partial word."""
    rng = np.random.default_rng(n)
    ids = rng.permutation(n).astype(np.int32)
    half, pairs = ids[: n // 2], ids[n // 2: n // 2 + 2 * (n // 8)]
    m = 8 * n + 1
    u = half[rng.integers(0, len(half), m)]
    v = half[rng.integers(0, len(half), m)]
    at = rng.choice(m, n // 8, replace=False)
    u[at], v[at] = pairs[0::2], pairs[1::2]
    want = oracle.labels(u, v, n)
    lab, st = cc.labels(put(u, dev), put(v, dev), n, return_stats=True)
    assert st["filter_used"] == 1
    assert np.array_equal(lab.cpu().numpy(), want)


def test_filtered_plan_without_a_giant(dev):
    """2,000 components of 100 vertices, their entries shuffled: no component
    holds an eighth of the samples, so nothing is filtered."""
    rng = np.random.default_rng(5)
    n, m = 200000, 1 << 21
    comp = rng.integers(0, 2000, m)
    u = (comp * 100 + rng.integers(0, 100, m)).astype(np.int32)
    v = (comp * 100 + rng.integers(0, 100, m)).astype(np.int32)
    lab, st = cc.labels(put(u, dev), put(v, dev), n, return_stats=True)
    assert st["hook"] == 1 and st["filter_used"] == 0
    assert np.array_equal(lab.cpu().numpy(), oracle.labels(u, v, n))


def test_racing_stores_settle(dev):
    """Regression: in the atomic-free Hook, workgroups on different XCDs store
    different parents to one slot; until the Multi-Jump after it stored every
    vertex, XCDs went on reading different values and most solves of these
    lists split a component.  Every one of many solves is compared."""
    for name, (u, v, n) in {
            "uniform 3n": (*graphgen.uniform_pairs(3 << 20, 1 << 20, seed=41, stream=0), 1 << 20),
            "uniform n": (*graphgen.uniform_pairs(1 << 20, 1 << 20, seed=42, stream=0), 1 << 20),
            "rmat20 3n": graphgen.rmat(20, 3, seed=43)}.items():
        want = torch.from_numpy(oracle.labels(u, v, n)).to(dev)
        du, dv = put(u, dev), put(v, dev)
        order = np.argsort(u, kind="stable")
        rp = torch.from_numpy(np.concatenate([[0], np.cumsum(np.bincount(u, minlength=n))])).to(dev)
        col = put(v[order], dev)
        out = torch.empty(n, dtype=torch.int32, device=dev)
        calls = {"csr hybrid": lambda: cc.labels_csr(rp, col, n, out=out,
                                                     options=cc.Options(hook="hybrid"))}
        for opt in (cc.Options(), cc.Options(hook="plain"), cc.Options(hook="hybrid"),
                    cc.Options(no_sync=True), cc.Options(hook="plain", host_loop="multijump"),
                    cc.Options(hook="plain", host_loop="jump")):
            calls[str(opt)] = lambda opt=opt: cc.labels(du, dv, n, out=out, options=opt)
        for what, call in calls.items():
            print("settle", name, what, flush=True)
            bad = 0
            for _ in range(15):
                out.fill_(-1)
                call()
                torch.cuda.synchronize()
                bad += not torch.equal(out, want)
            assert bad == 0, (name, what, bad)


# (n, entries per vertex): the hybrid plan's rules on one side and the other:
# no further rounds (sparse; more than 2^20 vertices), two further rounds, the
# last short list, lists with one chunk that has locality and one that has not
@pytest.mark.parametrize("n,m", [(40000, 30000), (40000, 44000), (1 << 20, 1 << 21),
                                 ((1 << 20) + 1, 1 << 21), (1 << 20, (1 << 22) - 1),
                                 (1 << 20, 1 << 22), (3000, 500000)])
def test_hybrid_plan(dev, n, m):
    u, v = graphgen.uniform_pairs(m, n, seed=n + m, stream=0)
    path = np.arange(n - 1, dtype=np.int32)
    lists = {"uniform": (u, v), "half a path": (np.concatenate([path, u[: m // 2]]),
                                                np.concatenate([path + 1, v[: m // 2]]))}
    hub = u.copy()
    hub[: m // 2] = n - 1  # half of the entries share an endpoint, the largest id
    lists["hub"] = (hub, v)
    for name, (a, b) in lists.items():
        want = oracle.labels(a, b, n)
        for offset in (0, 2):
            da, db = put(a, dev, offset), put(b, dev, offset)
            for opt in (cc.Options(), cc.Options(hook="hybrid", path_halving="off"),
                        cc.Options(no_sync=True)):
                print("hybrid", n, m, name, offset, opt.no_sync, flush=True)
                out = torch.full((n,), -7, dtype=torch.int32, device=dev)
                cc.labels(da, db, n, out=out, options=opt)
                torch.cuda.synchronize()
                assert np.array_equal(out.cpu().numpy(), want), (name, opt)
        if m < 1 << 22:
            out.fill_(-7)
            cc.labels_noalloc(da, db, n, out=out)
            assert np.array_equal(out.cpu().numpy(), want), name
    u[m - 1] = n
    with pytest.raises(cc.CCError) as ei:
        cc.labels(put(u, dev), put(v, dev), n)
    assert ei.value.code == cc.CC_ERR_RANGE


def to_csr(u, v, n):
    order = np.argsort(u, kind="stable")
    rp = np.zeros(n + 1, dtype=np.int64)
    np.cumsum(np.bincount(u, minlength=n), out=rp[1:])
    return rp, v[order].astype(np.int32)


# The CSR plans' sizes on one side and the other: part of a tile of 1,024
# entries, one tile, the last hybrid and the first filtered list, the last
# bitmap in LDS and the first one outside; a ragged end throughout
@pytest.mark.parametrize("n,m", [(1, 0), (70, 5), (100, 1023), (100, 1024), (5000, 40001),
                                 (100000, (1 << 20) - 1), (100000, (1 << 20) + 2),
                                 (1 << 20, (1 << 23) + 3), ((1 << 20) + 1, (1 << 23) + 9)])
def test_csr_plans(dev, n, m):
    u, v = graphgen.uniform_pairs(m, n, seed=n + m, stream=0)
    half = m // 2
    u2, v2 = np.concatenate([u[:half], v[:half]]), np.concatenate([v[:half], u[:half]])
    far = n - 1 - n // 4  # rows n // 4 .. are empty but the last: tiles of empty rows
    lists = {"uniform": (u, v, False), "both orientations": (u2, v2, True),
             "empty rows": (np.where(u < n // 4, u, n - 1), np.where(v < n // 4, v, far), False),
             # parts of 8 vertices: no giant, the filter stays off
             "small parts": (u, (u & ~7) + (v & 7).clip(max=(n - 1) & 7), False)}
    for name, (a, b, sym) in lists.items():
        b = np.minimum(b, n - 1).astype(np.int32)
        want = oracle.labels(a, b, n)
        rp, col = to_csr(a, b, n)
        drp = torch.from_numpy(rp).to(dev)
        for offset in (0, 1):
            dcol = put(col, dev, offset)
            for opt in (cc.Options(), cc.Options(path_halving="off"), cc.Options(no_sync=True),
                        cc.Options(symmetric=sym)):
                print("csr", n, m, name, offset, opt.no_sync, opt.symmetric, flush=True)
                out = torch.full((n,), -7, dtype=torch.int32, device=dev)
                cc.labels_csr(drp, dcol, n, out=out, options=opt)
                torch.cuda.synchronize()
                assert np.array_equal(out.cpu().numpy(), want), (name, opt)
    if m:
        for at, value in ((0, n), (m // 2, -1), (m - 1, n)):
            wrong = col.copy()
            wrong[at] = value
            with pytest.raises(cc.CCError) as ei:
                cc.labels_csr(drp, put(wrong, dev), n)
            assert ei.value.code == cc.CC_ERR_RANGE
        for at, value in ((0, 1), (n, m - 1), (n // 2, m + 5), (n // 2, -3)):
            wrong = rp.copy()
            wrong[at] = value
            with pytest.raises(cc.CCError) as ei:
                cc.labels_csr(torch.from_numpy(wrong).to(dev), put(col, dev), n)
            assert ei.value.code == cc.CC_ERR_RANGE


# Regression: lists with fewer than 8 entries per vertex or 2^20 entries took
# the hybrid plan past these options.  Rows of every kind: even ones, long
# empty ranges (a tile's row window is more than the LDS holds), hubs.
def test_csr_segment_options_get_segments(dev):
    rng = np.random.default_rng(11)
    hub = np.concatenate([np.full(30000, 17, np.int32), np.arange(9000, dtype=np.int32)])
    lists = {"uniform": (*graphgen.uniform_pairs(300000, 100000, seed=6, stream=0), 100000),
             "empty rows": (*graphgen.uniform_pairs(30000, 400000, seed=7, stream=0), 400000),
             "hub": (hub, rng.integers(0, 9000, len(hub)).astype(np.int32), 9000)}
    for name, (u, v, n) in lists.items():
        want = oracle.labels(u, v, n)
        rp, col = to_csr(u, v, n)
        drp, dcol = torch.from_numpy(rp).to(dev), put(col, dev, 1)
        for opt, segments in ((cc.Options(segments=3), 3), (cc.Options(filter="giant", segments=8), 8),
                              (cc.Options(filter="giant", segments=12, filter_after=2,
                                          path_halving="off"), 12),
                              (cc.Options(filter="off"), max(1, int(len(u) / n + 0.5)))):
            print("csr segments", name, opt, flush=True)
            lab, st = cc.labels_csr(drp, dcol, n, options=opt, return_stats=True)
            assert np.array_equal(lab.cpu().numpy(), want), (name, opt)
            assert (st["hook"], st["segments"]) == (1, segments), (name, opt)
        assert cc.labels_csr(drp, dcol, n, return_stats=True)[1]["hook"] == 3


def test_csr_capture_needs_no_memory(dev):
    """Inside a capture the plans that need more scratch than is there give way
    to the one that needs none; every replay is right."""
    n, m = 1 << 19, 3 << 19
    u, v = graphgen.uniform_pairs(m, n, seed=5, stream=0)
    want = torch.from_numpy(np.asarray(oracle.labels(u, v, n), dtype=np.int32)).to(dev)
    rp, col = to_csr(u, v, n)
    drp, dcol = torch.from_numpy(rp).to(dev), put(col, dev)
    out = torch.empty(n, dtype=torch.int32, device=dev)
    stream = torch.cuda.Stream()
    opt = cc.Options(no_sync=True)
    with torch.cuda.stream(stream):  # a small call: the stream's smallest scratch
        cc.labels_csr(torch.zeros(2, dtype=torch.int64, device=dev), dcol[:0], 1, options=opt, stream=stream)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=stream):
        cc.labels_csr(drp, dcol, n, out=out, options=opt, stream=stream)
    for _ in range(3):
        out.fill_(-1)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want)


def test_csr_capture_keeps_the_filter(dev):
    """Regression: inside a capture with too little scratch for the automatic
    filtered plan but room for the bitmap, a dense adjacency ran unfiltered; an
    explicit hybrid plan ran as another one instead of being refused."""
    u, v, n = graphgen.rmat(18, 8, seed=18, symmetrize=True)
    want = torch.from_numpy(np.asarray(oracle.labels(u, v, n), dtype=np.int32)).to(dev)
    rp, col = to_csr(u, v, n)
    drp, dcol = torch.from_numpy(rp).to(dev), put(col, dev)
    out = torch.empty(n, dtype=torch.int32, device=dev)
    stream = torch.cuda.Stream()
    opt = cc.Options(no_sync=True)
    with torch.cuda.stream(stream):  # a small call: the stream's smallest scratch
        cc.labels_csr(torch.zeros(2, dtype=torch.int64, device=dev), dcol[:0], 1, options=opt, stream=stream)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=stream):
        _, st = cc.labels_csr(drp, dcol, n, out=out, options=opt, stream=stream, return_stats=True)
        with pytest.raises(cc.CCError) as ei:
            cc.labels_csr(drp, dcol, n, out=out, options=cc.Options(no_sync=True, hook="hybrid"),
                          stream=stream)
    assert ei.value.code == cc.CC_ERR_NOMEM
    # segments of n / 16 entries, launched by growing numbers of them
    assert st["hook"] == 1 and st["segments"] == 16 * 16 and st["hook_launches"] < 16
    for _ in range(3):
        out.fill_(-1)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want)


# Graphs of a list that leave the LDS launch: none, one, two among small ones,
# and the sparse and dense graphs above the LDS's vertices
@pytest.mark.parametrize("sizes", [[(65536, 786431), (300, 900)],
                                   [(65536, 786432), (300, 900), (40, 0)],
                                   [(1, 800000), (2000, 1 << 20), (5000, 700000), (65536, 65536)],
                                   [(65536, 1 << 21), (65537, 65537), (65537, (1 << 21) + 1),
                                    (1 << 20, 1 << 22), (70000, 0), (0, 0)]])
def test_list_routes(dev, sizes):
    lists = [graphgen.uniform_pairs(m, max(n, 1), seed=n + m, stream=0) for n, m in sizes]
    want = [oracle.labels(u, v, n) for (u, v), (n, m) in zip(lists, sizes)]
    graphs = [(put(u, dev), put(v, dev), n) for (u, v), (n, m) in zip(lists, sizes)]
    for opt in (cc.Options(), cc.Options(segments=1), cc.Options(block=512), cc.Options(path_halving="off")):
        print("list", sizes, opt.segments, opt.block, flush=True)
        for got, lab in zip(cc.labels_list(graphs, options=opt), want):
            assert np.array_equal(got.cpu().numpy(), lab), opt
    stream = torch.cuda.Stream()
    stream.wait_stream(torch.cuda.current_stream())
    for rep in range(3):
        got = cc.labels_list(graphs, options=cc.Options(graph=True), stream=stream)
        for g, lab in zip(got, want):
            assert np.array_equal(g.cpu().numpy(), lab), rep
    # room for every request's edges and labels and little more: workspaces
    # are waited for or done without
    need = max(8 * m + 4 * n for n, m in sizes)
    for extra in (200 << 10, 64 << 20):
        with cc.Server(device_bytes=need + extra, workers=2, max_batch=8) as srv:
            tickets = [srv.submit(u, v, n) for u, v, n in graphs if n <= 65536 or extra > 1 << 20]
            kept = [lab for lab, (u, v, n) in zip(want, graphs) if n <= 65536 or extra > 1 << 20]
            for t, lab in zip(tickets, kept):
                got, info = srv.wait(t)
                assert np.array_equal(got.cpu().numpy(), lab)
    for i, (n, m) in enumerate(sizes):
        if m:
            bad = lists[i][1].copy()
            bad[m - 1] = n
            wrong = list(graphs)
            wrong[i] = (graphs[i][0], put(bad, dev), n)
            with pytest.raises(cc.CCError) as ei:
                cc.labels_list(wrong)
            assert ei.value.code == cc.CC_ERR_RANGE


def band(n, b):
    """Every vertex and the b ids on either side of it, in the order of the rows."""
    d = np.array([k for k in range(-b, b + 1) if k], dtype=np.int64)
    u = np.repeat(np.arange(n), 2 * b)
    v = u + np.tile(d, n)
    keep = (v >= 0) & (v < n)
    return u[keep].astype(np.int32), v[keep].astype(np.int32)


def median_us(call, passes=7):
    call()
    times = []
    for _ in range(passes):
        torch.cuda.synchronize()
        t = time.perf_counter()
        call()
        torch.cuda.synchronize()
        times.append((time.perf_counter() - t) * 1e6)
    return sorted(times)[passes // 2]


# Lists that leave chains of up to n levels: paths in rising, falling and
# random order at the sizes of the LDS solver (32- and 16-bit slots in batches),
# the window rounds and the Multi-Jump with two and four vertices per thread;
# bands in the order of their rows for the filtered plans with and without
# prefix rounds and the CSR plan.  Regression: the Multi-Jumps walked a chain one
# load at a time (5 to 340 times as long as the same graph takes with its ids
# permuted).  4 times is allowed; an exact pass each.  The last one has more
# vertices than the Multi-Jump's resident workgroups take at a time (8.4 s
# where they strode over the vertices, 1.6 ms now).
@pytest.mark.parametrize("what", ["path 1000", "path 32768", "path 50000", "path %d" % (1 << 20),
                                  "falling path %d" % (1 << 22), "shuffled path 32768",
                                  "shuffled path %d" % (1 << 21), "band5 %d" % (1 << 18),
                                  "band5 %d" % (1 << 19), "band5 %d" % (1 << 21),
                                  "csr band5 %d" % (1 << 21), "batch 32768", "batch 60000",
                                  "shuffled path %d" % (1 << 24)])
def test_chains(dev, what):
    kind, n = what.rsplit(" ", 1)
    n = int(n)
    rng = np.random.default_rng(n)
    if "band5" in kind:
        u, v = band(n, 5)
    else:
        u, v = np.arange(n - 1, dtype=np.int32), np.arange(1, n, dtype=np.int32)
    if kind == "falling path":
        u, v = u[::-1], v[::-1]
    if kind == "shuffled path":
        order = rng.permutation(len(u))
        u, v = u[order], v[order]
    perm = rng.permutation(n).astype(np.int32)
    times = []
    for a, b in ((u, v), (perm[u], perm[v])):
        if kind.startswith("csr"):
            rp, col = to_csr(a, b, n)
            drp, dcol = torch.from_numpy(rp).to(dev), put(col, dev)
            out = torch.empty(n, dtype=torch.int32, device=dev)
            call = lambda: cc.labels_csr(drp, dcol, n, out=out)  # noqa: E731
        elif kind == "batch":
            count = 5
            du, dv = put(np.tile(a, count), dev), put(np.tile(b, count), dev)
            vo, eo = np.arange(count + 1) * n, np.arange(count + 1) * len(a)
            out = torch.empty(count * n, dtype=torch.int32, device=dev)
            call = lambda: cc.labels_batch(du, dv, vo, eo, out=out)  # noqa: E731
        else:
            du, dv = put(a, dev), put(b, dev)
            out = torch.empty(n, dtype=torch.int32, device=dev)
            call = lambda: cc.labels(du, dv, n, out=out)  # noqa: E731
        for _ in range(5):
            out.fill_(-1)
            call()
            torch.cuda.synchronize()
            assert int(torch.count_nonzero(out)) == 0, what  # one component each
        times.append(median_us(call))
    print("chains", what, times, flush=True)
    assert times[0] <= 4 * times[1], (what, times)


def test_contracting_hook_spreads_over_the_roots(dev):
    """Regression: the workgroups of the contracting hook met on each root's
    word at the same time (0.86 times the time of the Atomic-Hook by segments
    on these adjacencies, 0.54 to 0.60 since; half-way is allowed)."""
    n, m = 200000, 600000
    times = np.zeros(2)
    for seed in (1, 2, 3):
        u, v = graphgen.uniform_pairs(m, n, seed=seed, stream=0)
        rp, col = to_csr(np.concatenate([u, v]), np.concatenate([v, u]), n)
        drp, dcol = torch.from_numpy(rp).to(dev), put(col, dev)
        out = torch.empty(n, dtype=torch.int32, device=dev)
        want = oracle.labels(u, v, n)
        for k, opt in enumerate((cc.Options(), cc.Options(hook="atomic"))):
            times[k] += median_us(lambda: cc.labels_csr(drp, dcol, n, out=out, options=opt), passes=15)
            assert np.array_equal(out.cpu().numpy(), want)
    print("contract", times, flush=True)
    assert times[0] <= 0.72 * times[1], times


def cliques(count, size):
    """Cliques of consecutive ids, their pairs in order."""
    i, j = np.triu_indices(size, 1)
    at = np.arange(count)[:, None] * size
    return (at + i).ravel().astype(np.int32), (at + j).ravel().astype(np.int32)


# Dense lists whose consecutive entries touch nearby ids.  Regression: the part
# of such a list that the filtered plan starts with holds no giant, and the
# launches after it hooked every entry (3.2 to 8.8 times as long as the hybrid
# plan; 1.2 to 1.9 since, 2.5 is allowed).  With them, sizes of each chunk length
# of the windows, a list that is two thirds such entries, and one without.
@pytest.mark.parametrize("what", ["cliques 2000x60", "cliques 10x800", "band 200000", "band 524288",
                                  "mixed", "random"])
def test_dense_lists_with_locality(dev, what):
    kind, _, size = what.partition(" ")
    rng = np.random.default_rng(17)
    if kind == "cliques":
        count, k = map(int, size.split("x"))
        n, (u, v) = count * k, cliques(count, k)
    else:
        n = int(size or 200000)
        u, v = band(n, 9) if kind == "band" else band(n, 6)
        if kind != "band":
            at = rng.permutation(len(u))[: len(u) // 3] if kind == "mixed" else np.arange(len(u))
            u[at], v[at] = rng.integers(0, n, (2, len(at)))
    want = oracle.labels(u, v, n)
    windows = kind in ("cliques", "band")
    for offset in (0, 1):
        du, dv = put(u, dev, offset), put(v, dev, offset)
        for opt in (cc.Options(), cc.Options(path_halving="off"), cc.Options(graph=True)):
            print("dense", what, offset, opt.path_halving, flush=True)
            for _ in range(4):
                out = torch.full((n + 1,), -7, dtype=torch.int32, device=dev)[1:]
                _, st = cc.labels(du, dv, n, out=out, options=opt, return_stats=True,
                                  stream=torch.cuda.Stream() if opt.graph else None)
                assert np.array_equal(out.cpu().numpy(), want), opt
            assert st["hook"] == 1 and st["filter_used"] == (0 if windows else 1)
    if windows:
        times = [median_us(lambda: cc.labels(du, dv, n, out=out, options=o), 15)
                 for o in (cc.Options(), cc.Options(hook="hybrid"))]
        print("dense times", what, times, flush=True)
        assert times[0] <= 2.5 * times[1], times
        listed = cc.labels_list([(du, dv, n), (du, dv, n)])
        assert all(np.array_equal(x.cpu().numpy(), want) for x in listed)
    for at in (0, len(u) // 2, len(u) - 1):
        keep, v[at] = v[at], n
        with pytest.raises(cc.CCError) as ei:
            cc.labels(du, put(v, dev), n)
        assert ei.value.code == cc.CC_ERR_RANGE
        v[at] = keep


def test_few_dense_graphs_take_two_segments(dev):
    """Regression: of a few graphs of four to eight entries per vertex each ran
    one segment (164 us for five of 60,000 vertices, 150 with two)."""
    n, count = 60000, 5
    u, v = graphgen.uniform_pairs(4 * n, n, seed=9, stream=0)
    du, dv = put(np.tile(u, count), dev), put(np.tile(v, count), dev)
    vo, eo = np.arange(count + 1) * n, np.arange(count + 1) * len(u)
    want = np.tile(oracle.labels(u, v, n), count)
    out = torch.empty(count * n, dtype=torch.int32, device=dev)
    times = {}
    for k in (0, 2) * 3:
        call = lambda: cc.labels_batch(du, dv, vo, eo, out=out, options=cc.Options(segments=k))  # noqa: E731
        times[k] = min(times.get(k, 1e9), median_us(call, 15))
        assert np.array_equal(out.cpu().numpy(), want)
    print("segments", times, flush=True)
    assert times[0] <= 1.05 * times[2], times


# The last adjacencies solved by one workgroup in LDS and the first ones past
# them, in a capture on a stream with the smallest scratch too
@pytest.mark.parametrize("n,m", [(1, 0), (1, 5), (300, 130472), (32768, 65536), (32768, 65537),
                                 (32769, 100)])
def test_small_csr(dev, n, m):
    u, v = graphgen.uniform_pairs(m, n, seed=n + m, stream=0)
    want = torch.from_numpy(np.asarray(oracle.labels(u, v, n), dtype=np.int32)).to(dev)
    rp, col = to_csr(u, v, n)
    drp = torch.from_numpy(rp).to(dev)
    stream = torch.cuda.Stream()
    empty = torch.zeros(2, dtype=torch.int64, device=dev)
    for offset in (0, 1):
        dcol = put(col, dev, offset)
        out = torch.full((n + 1,), -7, dtype=torch.int32, device=dev)[1:]
        for opt in (cc.Options(), cc.Options(path_halving="off"), cc.Options(profile=True)):
            out.fill_(-7)
            cc.labels_csr(drp, dcol, n, out=out, options=opt)
            assert torch.equal(out, want), opt
        with torch.cuda.stream(stream):
            cc.labels_csr(empty, dcol[:0], 1, options=cc.Options(no_sync=True), stream=stream)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=stream):
            cc.labels_csr(drp, dcol, n, out=out, options=cc.Options(no_sync=True), stream=stream)
        for _ in range(3):
            out.fill_(-1)
            torch.cuda.synchronize()
            g.replay()
            torch.cuda.synchronize()
            assert torch.equal(out, want)
    if m:
        for wrong in (np.where(np.arange(len(col)) == m // 2, n, col),
                      np.where(np.arange(len(col)) == 0, -1, col)):
            with pytest.raises(cc.CCError) as ei:
                cc.labels_csr(drp, put(wrong, dev), n)
            assert ei.value.code == cc.CC_ERR_RANGE
        rp[n] += 1
        for opt in (cc.Options(), cc.Options(no_sync=True)):
            with pytest.raises(cc.CCError) as ei:
                cc.labels_csr(torch.from_numpy(rp).to(dev), dcol, n, options=opt)
                torch.cuda.synchronize()
                cc.stream_status()
            assert ei.value.code == cc.CC_ERR_RANGE


def test_small_csr_latency(dev):
    """Regression: the hybrid plan's chain of launches on the smallest
    adjacencies (1.4 to 1.7 times the Atomic-Hook by segments)."""
    for n in (30, 1000, 15000):
        u, v = np.arange(n - 1, dtype=np.int32), np.arange(1, n, dtype=np.int32)
        if n == 15000:
            u[:] = 0  # a star
        rp, col = to_csr(np.concatenate([u, v]), np.concatenate([v, u]), n)
        drp, dcol = torch.from_numpy(rp).to(dev), put(col, dev)
        times = [median_us(lambda: cc.labels_csr(drp, dcol, n, options=o), 31)
                 for o in (cc.Options(), cc.Options(hook="atomic"))]
        print("small csr", n, times, flush=True)
        assert times[0] <= 1.1 * times[1], (n, times)


# Each side of the limits of the automatic choice: the plan that runs, its
# edge passes and the segments it reports.
def test_automatic_plans(dev):
    def pairs(n, m):
        return graphgen.uniform_pairs(m, n, seed=n % 97, stream=0)

    def stats(n, m, csr, **opt):
        u, v = pairs(n, m)
        want = oracle.labels(u, v, n)
        if csr:
            rp, col = to_csr(u, v, n)
            lab, st = cc.labels_csr(torch.from_numpy(rp).to(dev), put(col, dev), n,
                                    options=cc.Options(**opt), return_stats=True)
        else:
            lab, st = cc.labels(put(u, dev), put(v, dev), n, options=cc.Options(**opt), return_stats=True)
        assert np.array_equal(lab.cpu().numpy(), want), (n, m, csr)
        print("automatic plan", n, m, csr, opt, st["hook"], st["segments"], st["filter_used"],
              st["hook_launches"], flush=True)
        return st["hook"], st["segments"], st["filter_used"], st["hook_launches"]

    # (hook, segments, filter used, edge passes); 1 Atomic-Hook, 2 atomic-free, 3 hybrid
    assert stats(32768, 65536, False) == (2, 0, 0, 1)       # one workgroup in LDS
    assert stats(32768, 65537, False) == (3, 0, 0, 4)       # window round, two more, contraction
    assert stats(32769, 20000, False) == (3, 0, 0, 2)       # no further round
    assert stats(100000, 600000, False) == (3, 0, 0, 3)     # one further round
    assert stats(1 << 18, (1 << 21) - 1, False)[0] == 3
    # four rounds over the first n entries, then up to 3 n and the rest
    assert stats(1 << 18, 1 << 21, False) == (1, 2, 1, 6)
    assert stats(1 << 19, 1 << 22, False) == (1, 2, 1, 6)
    assert stats(5000, 1 << 21, False) == (1, 4, 1, 8)
    # above 2^19 vertices segments of n / 16 entries: 1, 2, 8, 32, 128 and 85 of them
    assert stats((1 << 19) + 1, 1 << 23, False) == (1, 256, 1, 6)
    assert stats(1 << 20, (1 << 22) - 1, False)[3] == 4
    assert stats(1 << 20, 1 << 22, False)[3] == 5            # and the pairs of long lists
    assert stats(32768, 65536, True) == (3, 0, 0, 1)
    assert stats(32768, 65537, True) == (3, 0, 0, 4)
    assert stats(1 << 17, (1 << 20) - 1, True)[0] == 3
    assert stats(1 << 17, 1 << 20, True) == (1, 1, 1, 3)
    assert stats(1 << 17, 1 << 20, True, segments=8)[:2] == (1, 8)


# Rows of up to several thousand entries that are not inside a giant: on both
# sides of the longest row that one lane marks (32), of a wave, of a tile of
# 1,024 entries; the filter off (64 equal components) and on (a giant beside
# them, in rows of its own and mixed with theirs).
@pytest.mark.parametrize("what", ["equal", "beside", "mixed"])
@pytest.mark.parametrize("offset", [0, 1])
def test_csr_long_rows(dev, what, offset):
    rng = np.random.default_rng(41)
    if what == "equal":
        n = 64 * 256
        rows = np.repeat(np.arange(n, dtype=np.int64), rng.integers(30, 60, n))
        u, v = rows, rows // 256 * 256 + rng.integers(0, 256, len(rows))
    else:
        size = 60000
        degrees = [31, 32, 33, 34, 63, 64, 65, 256, 1000, 1023, 1024, 1025, 3000, 5000]
        u, v = [rng.integers(0, size, 10 * size)], [rng.integers(0, size, 10 * size)]
        n = size
        for d in degrees:  # a star whose hub repeats its leaves, beside a component of such rows
            u += [np.full(d, n), np.repeat(n + 50 + np.arange(20), d // 2)]
            v += [n + 1 + np.arange(d) % 49, n + 50 + rng.integers(0, 20, 20 * (d // 2))]
            n += 70
        u, v = np.concatenate(u), np.concatenate(v)
        if what == "mixed":
            relabel = rng.permutation(n)
            u, v = relabel[u], relabel[v]
    u, v = np.concatenate([u, v]).astype(np.int32), np.concatenate([v, u]).astype(np.int32)
    assert len(u) >= 1 << 20 and len(u) >= 8 * n
    want = oracle.labels(u, v, n)
    rp, col = to_csr(u, v, n)
    drp, dcol = torch.from_numpy(rp).to(dev), put(col, dev, offset)
    for opt in (cc.Options(), cc.Options(symmetric=True), cc.Options(path_halving="off")):
        for _ in range(3):
            lab, st = cc.labels_csr(drp, dcol, n, options=opt, return_stats=True)
            assert np.array_equal(lab.cpu().numpy(), want), (what, opt)
        assert (st["hook"], st["segments"], st["filter_used"]) == (1, 1, int(what != "equal"))


# `out` one word past a 16-byte boundary, its neighbours untouched, on every
# automatic plan: further rounds, the pairs of long lists, both filtered plans
# of pair lists (bitmap in LDS, half of it, vertex table), both of CSR.
@pytest.mark.parametrize("n,m", [(100003, 300001), (1 << 20, (1 << 22) + 1), (1 << 18, (1 << 21) + 3),
                                 ((1 << 19) + 5, (1 << 22) + 77), (1400003, 11300001),
                                 (2700001, 21700001)])
@pytest.mark.parametrize("local", [False, True])
def test_unaligned_labels(dev, n, m, local):
    u, v = graphgen.uniform_pairs(m, n, seed=m % 89, stream=0)
    if local:  # consecutive entries touch nearby ids
        u = (np.arange(m, dtype=np.int64) * n // m).astype(np.int32)
        v = np.minimum(u + v % 5, n - 1).astype(np.int32)
    want = torch.from_numpy(np.asarray(oracle.labels(u, v, n), dtype=np.int32)).to(dev)
    du, dv = put(u, dev), put(v, dev)
    buf = torch.empty(n + 2, dtype=torch.int32, device=dev)
    for opt in (cc.Options(), cc.Options(hook="hybrid")):
        buf.fill_(-7)
        cc.labels(du, dv, n, out=buf[1:-1], options=opt)
        assert torch.equal(buf[1:-1], want) and buf[0] == -7 and buf[-1] == -7, opt
    if m < 1 << 22:
        rp, col = to_csr(u, v, n)
        drp, dcol = torch.from_numpy(rp).to(dev), put(col, dev)
        buf.fill_(-7)
        cc.labels_csr(drp, dcol, n, out=buf[1:-1])
        assert torch.equal(buf[1:-1], want) and buf[0] == -7 and buf[-1] == -7


# Long lists with locality: the compaction and the pairs, chosen and asked for
@pytest.mark.parametrize("what", ["grid", "band", "shuffled"])
def test_long_lists_with_locality(dev, what):
    if what == "grid":
        u, v, n = graphgen.grid(2000, 1990)
    else:
        n = 1 << 21
        u = np.repeat(np.arange(n, dtype=np.int32), 3)
        v = np.minimum(u + np.random.default_rng(3).integers(1, 9, len(u)), n - 1).astype(np.int32)
        if what == "shuffled":  # its entries in another order: the contracting hook
            order = np.random.default_rng(4).permutation(len(u))
            u, v = u[order], v[order]
    assert len(u) >= 1 << 22
    want = oracle.labels(u, v, n)
    for offset in (0, 1):
        du, dv = put(u, dev, offset), put(v, dev, offset)
        for opt in (cc.Options(), cc.Options(hook="hybrid"), cc.Options(hook="hybrid", path_halving="off")):
            for _ in range(3):
                lab, st = cc.labels(du, dv, n, options=opt, return_stats=True)
                assert np.array_equal(lab.cpu().numpy(), want), opt
            assert (st["hook"], st["hook_launches"]) == (3, 4), opt
