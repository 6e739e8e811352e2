"""A removed vertex with more than 2,048 candidate members (the h >= 4 peel
then counts its neighbours' out-neighbourhoods one by one): a hub that closes
one h-clique with one of many disjoint K_{h+1}.  The hub leaves first, with
core number 1, and every other vertex keeps core number C(h, h-1) = h."""
import numpy as np
import pytest

from paper_1906_00341_amd import dsd, synth

pytestmark = pytest.mark.gpu


def hub_graph(h, members):
    """Disjoint K_{h+1}, and a hub joined to h - 2 vertices of each (no h-clique) and h - 1 of the first (one)."""
    m, per = h + 1, h - 2
    k = -(-members // per)
    _, i, j = synth.complete_graph(m)
    at = np.arange(k, dtype=np.int64)[:, None] * m
    s, d = (at + i).ravel(), (at + j).ravel()
    near = np.concatenate([(at + np.arange(per)).ravel(), [per]])
    n = k * m + 1
    perm = np.random.default_rng(h).permutation(n)
    src, dst = np.concatenate([s, np.full(near.size, n - 1)]), np.concatenate([d, near])
    return n, perm[src].astype(np.int32), perm[dst].astype(np.int32), int(perm[n - 1])


@pytest.mark.parametrize("engine", ["0", "1"])
@pytest.mark.parametrize("h", [4, 5, 6])
@pytest.mark.parametrize("members", [2100, 4201])
def test_hub_leaves_with_one_clique(monkeypatch, h, members, engine):
    monkeypatch.setenv("DSD_TAIL_ENGINE", engine)
    n, s, d, hub = hub_graph(h, members)
    g = dsd.build_csr(n, s, d)
    core, km = dsd.clique_core(g, h)
    g.free()
    want = np.full(n, h, np.uint64)
    want[hub] = 1
    np.testing.assert_array_equal(core, want)
    assert km == h
