"""The clique tail (adjacency bitmaps, one workgroup per graph) against the
oracle and against the round kernels it replaces (DSD_TAIL_ENGINE=0), at the
sizes where its paths change: candidate sets of 64 / 65, 256 / 257, 512 / 513
and more than 4,096 members, frontiers beyond its candidate list, graphs on
both sides of the batch's workgroup sizes, widths that make it rebuild its
matrix.  Integers: equality, no tolerance."""
import numpy as np
import pytest

import oracle
from paper_1906_00341_amd import dsd, synth
from test_gpu_peel_hub import hub_graph

pytestmark = pytest.mark.gpu


def _dense(n, p, seed):
    rng = np.random.default_rng(seed)
    i, j = np.triu_indices(n, 1)
    keep = rng.random(i.size) < p
    return n, i[keep].astype(np.int32), j[keep].astype(np.int32)


def _cliques(sizes, seed=0):
    """Disjoint complete graphs of the given sizes, ids permuted."""
    s, d, at = [], [], 0
    for m in sizes:
        i, j = np.triu_indices(m, 1)
        s.append(i + at)
        d.append(j + at)
        at += m
    perm = np.random.default_rng(seed).permutation(at).astype(np.int32)
    return at, perm[np.concatenate(s)], perm[np.concatenate(d)]


def _core(monkeypatch, g, h, engine):
    monkeypatch.setenv("DSD_TAIL_ENGINE", engine)
    n, s, d = g
    gg = dsd.build_csr(n, s, d)
    core, km = dsd.clique_core(gg, h)
    st = gg.stats()
    mem, km2, dens = dsd.core_app(gg, h)
    pm, pd, pr, pb = dsd.peel_app(gg, h)
    gg.free()
    return core, km, st["peel_rounds"], st["peel_levels"], st["k4_tail_launches"], mem, km2, dens, pm, pd, pr, pb


def _same(a, b):
    for x, y in zip(a, b):
        if isinstance(x, np.ndarray):
            np.testing.assert_array_equal(x, y)
        else:
            assert x == y


CASES = {
    "dense40": (lambda: _dense(40, 0.6, 1), (4, 5, 6), True),
    "dense75": (lambda: _dense(75, 0.7, 2), (4, 5), True),
    "dense140": (lambda: _dense(140, 0.6, 3), (4, 5), True),
    "dense300": (lambda: _dense(300, 0.35, 4), (4, 5), True),
    "dense290": (lambda: _dense(290, 0.93, 5), (4,), False),
    "dense530": (lambda: _dense(530, 0.97, 6), (4,), False),
    "dense600": (lambda: _dense(600, 0.93, 7), (4,), False),
    "edges64": (lambda: _cliques([64, 65, 66, 67, 68]), (4, 5, 6), False),
    "edges256": (lambda: _cliques([255, 256, 257, 258, 259]), (4,), False),
    "edges512": (lambda: _cliques([511, 512, 513, 514, 515]), (4,), False),
    "mass": (lambda: _cliques([5] * 1000 + [6] * 900 + [7] * 3), (4, 5), True),
    "widths": (lambda: _cliques(list(range(5, 41)) * 28), (4, 6), False),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_single(monkeypatch, name):
    make, hs, with_oracle = CASES[name]
    g = make()
    for h in hs:
        new = _core(monkeypatch, g, h, "1")
        old = _core(monkeypatch, g, h, "0")
        assert new[4] > 0 and old[4] == 0, h
        _same(new[:4] + new[5:], old[:4] + old[5:])
        if with_oracle:
            core, km = oracle.Graph(*g).core_decomposition(h)
            np.testing.assert_array_equal(new[0], core)
            assert new[1] == km


@pytest.mark.parametrize("h", [4, 5, 6])
def test_hub_of_more_than_4096_members(monkeypatch, h):
    n, s, d, hub = hub_graph(h, 4201)
    new = _core(monkeypatch, (n, s, d), h, "1")
    old = _core(monkeypatch, (n, s, d), h, "0")
    _same(new[:4] + new[5:], old[:4] + old[5:])
    assert new[0][hub] == 1                # one clique, gone first


def test_rmat_rebuilds_its_matrix(monkeypatch):
    g = synth.rmat(scale=14, edge_factor=16, seed=5)
    for h in (4, 5):
        new = _core(monkeypatch, g, h, "1")
        old = _core(monkeypatch, g, h, "0")
        assert new[4] > 0
        _same(new[:4] + new[5:], old[:4] + old[5:])


@pytest.mark.parametrize("count", [3, 40])
def test_batch(monkeypatch, count):
    made = [_dense(30 + 9 * (i % 31), 0.5, 10 + i) for i in range(count)]
    made[1] = _cliques(list(range(5, 41)) * 28)                  # more vertices than the small workgroup takes
    made[2] = _cliques([5] * 500 + [6] * 400 + [7] * 3)          # frontiers beyond its candidate list
    hs = [4 + i % 3 if i > 2 else 4 for i in range(count)]
    out = {}
    for engine in ("1", "0"):
        monkeypatch.setenv("DSD_TAIL_ENGINE", engine)
        for op in ("core", "peel"):
            gs = [dsd.build_csr(*g) for g in made]
            outs = [np.zeros(g[0], np.uint64 if op == "core" else np.uint8) for g in made]
            res = dsd.batch_run(gs, hs, op, outs=outs)
            out[engine, op] = (outs, [(r["status"], r["kmax"], r["density"], r["peel_rounds"]) for r in res])
            for g in gs:
                g.free()
    for op in ("core", "peel"):
        assert out["1", op][1] == out["0", op][1]
        for a, b in zip(out["1", op][0], out["0", op][0]):
            np.testing.assert_array_equal(a, b)
