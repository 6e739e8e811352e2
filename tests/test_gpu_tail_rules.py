"""Where the clique tail takes over, and which rounds its workgroup keeps, by
the counts it reports; results against closed forms and the round kernels."""
from math import comb

import numpy as np
import pytest

from paper_1906_00341_amd import dsd
from test_gpu_clique_tail import _cliques

pytestmark = pytest.mark.gpu


def test_dense_vertices_stay_with_the_round_kernels():
    # h = 5, 16,341 vertices of degree 399 to 437 (a member's set costs the
    # tail's workgroup more than it keeps) behind 120 that leave first: the
    # tail waits for fewer vertices than the 15,000 that four rounds leave
    sizes = [6] * 20 + list(range(400, 439))
    n, s, d = _cliques(sizes)
    g = dsd.build_csr(n, s, d)
    core, km = dsd.clique_core(g, 5)
    st = g.stats()
    g.free()
    assert km == comb(437, 4)
    want = np.concatenate([np.full(m, comb(m - 1, 4), np.uint64) for m in sizes])
    np.testing.assert_array_equal(np.sort(core), np.sort(want))
    assert 0 < st["k4_tail_vertices"] < 14000
