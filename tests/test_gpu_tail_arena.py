"""The clique tail's large rounds with an arena that holds few of their
vertices (DSD_CT_ARENA_WORDS): those without room go back to their graph and
wait for the next sequence.  Against the round kernels; integers: equality."""
import numpy as np
import pytest

from paper_1906_00341_amd import dsd
from test_gpu_clique_tail import _cliques, _core, _dense, _same

pytestmark = pytest.mark.gpu

GRAPHS = {
    "cliques": lambda: _cliques([100, 130, 130, 131, 200, 257]),
    "dense": lambda: _dense(260, 0.7, 31),
}


@pytest.mark.parametrize("h", [4, 5, 6])
@pytest.mark.parametrize("name", sorted(GRAPHS))
def test_single(monkeypatch, name, h):
    g = GRAPHS[name]()
    roomy = _core(monkeypatch, g, h, "1")
    old = _core(monkeypatch, g, h, "0")
    monkeypatch.setenv("DSD_CT_ARENA_WORDS", "0")
    new = _core(monkeypatch, g, h, "1")
    _same(new[:4] + new[5:], old[:4] + old[5:])
    _same(roomy[:4] + roomy[5:], old[:4] + old[5:])
    if name == "cliques":                            # (a clique is one round of all its vertices)
        assert new[4] > roomy[4] > 0                 # sequences: some vertices waited


@pytest.mark.parametrize("h", [4, 5, 6])
def test_batch(monkeypatch, h):
    made = [_cliques([100, 131, 200]), _dense(220, 0.7, 32), _cliques([5] * 900 + [90, 120]), _dense(90, 0.6, 33),
            _cliques([257]), _dense(150, 0.8, 34)]
    got = {}
    for engine in ("1", "0"):
        monkeypatch.setenv("DSD_TAIL_ENGINE", engine)
        monkeypatch.setenv("DSD_CT_ARENA_WORDS", "0")
        for op in ("core", "peel"):
            gs = [dsd.build_csr(*g) for g in made]
            outs = [np.zeros(g[0], np.uint64 if op == "core" else np.uint8) for g in made]
            res = dsd.batch_run(gs, h, op, outs=outs)
            got[engine, op] = outs, [(r["status"], r["kmax"], r["density"], r["peel_rounds"]) for r in res]
            for g in gs:
                g.free()
    for op in ("core", "peel"):
        assert got["1", op][1] == got["0", op][1]
        for a, b in zip(got["1", op][0], got["0", op][0]):
            np.testing.assert_array_equal(a, b)
