"""A served request's memory beyond its footprint (the adjacency bitmaps of an
h >= 4 peel) comes out of the server's budget: refused where it does not fit,
given back when the request ends.  Results are those of the plain call."""
import numpy as np
import pytest

from paper_1906_00341_amd import dsd
from test_gpu_clique_tail import _cliques

pytestmark = pytest.mark.gpu

N, SRC, DST = _cliques(list(range(5, 61)) * 5)
FOOTPRINT = 160 * N + 192 * SRC.size


def _served(budget, count, h=4):
    srv = dsd.Server(budget, 8)
    got = []
    for _ in range(count):
        g = dsd.build_csr(N, SRC, DST)
        out = np.zeros(N, np.uint64)
        st, r = srv.wait(srv.submit(g, h, "core", out=out))
        assert st == 0 and r["status"] == 0
        dsd.clique_core(g, h)                        # kept by the request: its peel's figures
        got.append((out, r["kmax"], g.stats()["k4_tail_launches"]))
        g.free()
    srv.close()
    return got


def test_bitmaps_stay_within_the_budget():
    g = dsd.build_csr(N, SRC, DST)
    want, km = dsd.clique_core(g, 4)
    assert g.stats()["k4_tail_launches"] > 0
    g.free()
    # no smaller arena than 2^16 words: 64 KB never hold the bitmaps
    for out, k, launches in _served(FOOTPRINT + (64 << 10), 1):
        np.testing.assert_array_equal(out, want)
        assert k == km and launches == 0
    # room for one request's bitmaps at a time (8 (17 A^2 / 64 + 2^16) bytes): every one has them
    words = N * -(-N // 64)
    for out, k, launches in _served(FOOTPRINT + 8 * 18 * words + (32 << 20), 4):
        np.testing.assert_array_equal(out, want)
        assert k == km and launches > 0
