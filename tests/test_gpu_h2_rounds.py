"""The h = 2 round kernel against the oracle, at the row lengths where a
frontier vertex changes from 16 lanes to a whole wave (512), rounds whose
frontier is longer than a block's list of pushed vertices, batches and the
min-degree order.  Integers: equality, no tolerance."""
import numpy as np
import pytest

import oracle
from paper_1906_00341_amd import dsd, synth

pytestmark = pytest.mark.gpu


def _stars(sizes, spokes_joined):
    # hubs of the given degrees; consecutive leaves of a hub joined so that they outlive their first round
    src, dst, n = [], [], 0
    for d in sizes:
        leaf = np.arange(n + 1, n + 1 + d)
        src.append(np.full(d, n))
        dst.append(leaf)
        if spokes_joined:
            src.append(leaf[:-1])
            dst.append(leaf[1:])
        n += d + 1
    return n, np.concatenate(src).astype(np.int32), np.concatenate(dst).astype(np.int32)


GRAPHS = {
    "rows around 512": lambda: _stars([1, 15, 16, 17, 63, 64, 65, 511, 512, 513, 575, 576, 577, 2049, 5000], True),
    "leaves fall together": lambda: _stars([30000, 70000], False),
    "wheel spokes": lambda: _stars([40000], True),
    "path": lambda: (18000, np.arange(17999, dtype=np.int32), np.arange(1, 18000, dtype=np.int32)),
    "power law": lambda: synth.chung_lu(n=60000, avg_deg=14.0, beta=2.2, planted=2, plant_size=80, p=0.7, seed=2),
}


@pytest.mark.parametrize("name", list(GRAPHS))
@pytest.mark.parametrize("engine", ["0", "1"])
def test_core(monkeypatch, name, engine):
    monkeypatch.setenv("DSD_TAIL_ENGINE", engine)
    made = GRAPHS[name]()
    want, km = oracle.Graph(*made).core_decomposition(2)
    g = dsd.build_csr(*made)
    got, gkm = dsd.clique_core(g, 2)
    member, density, rounds, best = dsd.peel_app(g, 2)
    g.free()
    np.testing.assert_array_equal(got, want)
    assert gkm == km
    omember, odensity, orounds, obest = oracle.Graph(*made).peel_app(2)
    np.testing.assert_array_equal(np.asarray(member).astype(bool), omember)
    assert (density, rounds, best) == (odensity, orounds, obest)


def test_batch(monkeypatch):
    monkeypatch.setenv("DSD_TAIL_ENGINE", "0")
    made = [f() for f in GRAPHS.values()]
    gs = [dsd.build_csr(*m) for m in made]
    outs = [np.zeros(m[0], np.uint64) for m in made]
    res = dsd.batch_run(gs, 2, "core", outs=outs)
    for g in gs:
        g.free()
    for m, out, r in zip(made, outs, res):
        want, km = oracle.Graph(*m).core_decomposition(2)
        np.testing.assert_array_equal(out, want)
        assert r["kmax"] == km
