"""CSR build at the sizes where its kernels change: vertex degrees counted per
id range in LDS (large edge lists) against plain counting, id widths on both
sides of a power of two, and ids in hub order (one range split over
workgroups).  Integers: equality, no tolerance."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _degrees(n, s, d):
    keep = s != d
    lo, hi = np.minimum(s, d)[keep].astype(np.int64), np.maximum(s, d)[keep].astype(np.int64)
    key = np.unique(lo * n + hi)
    return np.bincount(key // n, minlength=n) + np.bincount(key % n, minlength=n), key


def _check(n, s, d):
    import torch
    from paper_1906_00341_amd import dsd
    want, key = _degrees(n, s, d)
    g = dsd.build_csr(n, torch.from_numpy(s).cuda(), torch.from_numpy(d).cuda())
    assert g.info() == (n, key.size)
    deg, m = dsd.clique_degrees(g, 2)
    assert m == key.size
    assert np.array_equal(deg.astype(np.int64), want)
    st = g.stats()
    # the orientation: out-degrees by (degree, id) rank
    rank = np.empty(n, np.int64)
    rank[np.lexsort((np.arange(n), want))] = np.arange(n)
    a, b = key // n, key % n
    low = np.where(rank[a] < rank[b], a, b)
    out = np.bincount(low, minlength=n)
    assert st["w2"] == int(((want - out) * out).sum()) and st["s2"] == int((want * out).sum())
    g.free()


@pytest.mark.parametrize("n", [300, 511, 512, 65535, 65536, 300007])
@pytest.mark.parametrize("pairs", [1, 4096, (1 << 18) + 5, 700001])
def test_degrees_and_wedges(n, pairs):
    rng = np.random.default_rng(n + pairs)
    s = rng.integers(0, n, pairs).astype(np.int32)
    d = (rng.integers(0, n, pairs) * rng.random(pairs) ** 3).astype(np.int32)
    _check(n, s, d)


def test_hub_order_ids():
    # the 512 vertices of one id range hold more than 2^20 ends, most vertices none
    n = 100000
    rng = np.random.default_rng(3)
    s = np.repeat(np.arange(512, dtype=np.int32), 2600)
    d = rng.integers(0, n // 2, s.size).astype(np.int32)
    _check(n, s, d)
    _check(n, n - 1 - s, n - 1 - d)
