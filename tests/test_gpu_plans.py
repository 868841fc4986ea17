"""The automatic plan's paths at the sizes where its rules change and its
kernels have edges, against the CPU oracle (integer labels with one correct
answer: every comparison is bit-exact)."""
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
