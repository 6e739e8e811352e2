"""Values read back through the pinned buffer against plain copies, by way of
calls whose results pass through it: a level table longer than the part that
comes along, several threads (a buffer each), and root lists at the edges of a
workgroup's 4,096 roots.  Integers: equality."""
import threading

import numpy as np
import pytest

import oracle
from paper_1906_00341_amd import dsd, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 2, 4095, 4096, 4097, 12289])
@pytest.mark.parametrize("h", [3, 4])
def test_degrees_at_the_edges_of_a_workgroup(n, h):
    made = synth.chung_lu(n=n, avg_deg=8.0, beta=2.3, planted=1, plant_size=30, p=0.7, seed=n) if n > 100 \
        else synth.complete_graph(n)
    g = dsd.build_csr(*made)
    out, mu = dsd.clique_degrees(g, h)
    fixed, fmu = dsd.clique_degrees_noalloc(g, h)
    want, wmu = oracle.Graph(*made).clique_degrees(h)
    g.free()
    np.testing.assert_array_equal(fixed, want)
    assert fmu == wmu
    np.testing.assert_array_equal(out, want)
    assert mu == wmu


def test_threads_read_back_at_the_same_time():
    made = [synth.chung_lu(n=3000 + 17 * i, avg_deg=10.0, beta=2.3, planted=1, plant_size=40, p=0.7, seed=i)
            for i in range(6)]
    want = [oracle.Graph(*m).core_decomposition(3) for m in made]
    got = [None] * len(made)

    def work(i):
        for _ in range(3):
            g = dsd.build_csr(*made[i])
            got[i] = dsd.clique_core(g, 3)
            g.free()

    ts = [threading.Thread(target=work, args=(i,)) for i in range(len(made))]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    for (core, km), (out, gkm) in zip(want, got):
        np.testing.assert_array_equal(out, core)
        assert gkm == km


def test_a_level_table_beyond_the_part_that_comes_along():
    made = synth.chung_lu(n=3000, avg_deg=200.0, beta=2.5, planted=0, plant_size=10, p=0.8, seed=5)
    core, km = oracle.Graph(*made).core_decomposition(3)
    assert len(np.unique(core)) > 512
    g = dsd.build_csr(*made)
    out, gkm = dsd.clique_core(g, 3)
    levels = g.stats()["peel_levels"]
    g.free()
    np.testing.assert_array_equal(out, core)
    assert gkm == km
    assert levels >= len(np.unique(core[core > 0]))
