"""One root whose out-neighbourhood is a sparse random graph, at the
out-degrees of the bins that complete graphs alone had met (all rows of a
complete graph are alike): h = 4 from 769 to 1,089 out-neighbours, h = 6 from
257 to 513.  Against the oracle; integers: equality, no tolerance."""
import numpy as np
import pytest

import oracle
from paper_1906_00341_amd import dsd
from test_gpu_enum_rows import _hub_pair

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("h,k", [(4, 769), (4, 1000), (4, 1088), (4, 1089), (6, 257), (6, 300), (6, 512), (6, 513)])
def test_one_root_against_oracle(h, k):
    # some 60 or 110 neighbours inside for each of the root's: thousands of cliques, and a quick oracle
    n, s, d = _hub_pair(k, (60 if h == 4 else 110) / k, k)
    want, mu_o = oracle.Graph(n, s, d).clique_degrees(h)
    g = dsd.build_csr(n, s, d)
    deg, mu = dsd.clique_degrees(g, h)
    g.free()
    assert mu == mu_o > 0
    np.testing.assert_array_equal(deg, want)
