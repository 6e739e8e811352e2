"""The tail engine over a batch (a workgroup per graph) and in the min-degree
order, against the round kernels (DSD_TAIL_ENGINE=0) and the oracle, at the
vertex counts where its workgroups change (2,048, 4,096, 16,384) and beyond
them.  Integers: equality, no tolerance."""
import numpy as np
import pytest

import oracle
from paper_1906_00341_amd import dsd, synth

pytestmark = pytest.mark.gpu

SIZES = [1, 5, 300, 2047, 2048, 2049, 4096, 4097, 16383, 16384, 16385, 21000]


def _graph(n, seed):
    if n < 300:
        return synth.complete_graph(n)
    return synth.chung_lu(n=n, avg_deg=12.0, beta=2.3, planted=2, plant_size=40, p=0.6, seed=seed)


def _run(made, h, op):
    gs = [dsd.build_csr(n, s, d) for n, s, d in made]
    outs = [np.zeros(max(n, 1), np.uint64 if op == "core" else np.uint8) for n, _, _ in made]
    res = dsd.batch_run(gs, h, op, outs=outs)
    for g in gs:
        g.free()
    return outs, [(r["status"], r["kmax"], r["density"], r["members"], r["peel_rounds"], r["num_cliques"]) for r in res]


@pytest.mark.parametrize("op", ["core", "peel"])
@pytest.mark.parametrize("h", [2, 3])
@pytest.mark.parametrize("sizes", [SIZES, [1500] * 40, [17000, 90]])
def test_batch_engine_matches_rounds(monkeypatch, h, op, sizes):
    made = [_graph(n, 3 + i) for i, n in enumerate(sizes)]
    monkeypatch.setenv("DSD_TAIL_ENGINE", "1")
    new = _run(made, h, op)
    monkeypatch.setenv("DSD_TAIL_ENGINE", "0")
    old = _run(made, h, op)
    assert new[1] == old[1]
    for a, b in zip(new[0], old[0]):
        np.testing.assert_array_equal(a, b)
    if op == "core":
        for i in (0, len(made) - 1):
            core, km = oracle.Graph(*made[i]).core_decomposition(h)
            np.testing.assert_array_equal(new[0][i][:made[i][0]], core)
            assert new[1][i][1] == km


@pytest.mark.parametrize("h", [2, 3])
@pytest.mark.parametrize("n", [700, 16384, 20000])
def test_peel_app_engine_matches_rounds(monkeypatch, h, n):
    made = _graph(n, 11)
    got = {}
    for engine, heavy in (("1", None), ("1", "0"), ("0", None)):
        monkeypatch.setenv("DSD_TAIL_ENGINE", engine)
        if heavy is None:
            monkeypatch.delenv("DSD_TE_GRID_PAIRS", raising=False)
        else:
            monkeypatch.setenv("DSD_TE_GRID_PAIRS", heavy)
        g = dsd.build_csr(*made)
        got[engine, heavy] = dsd.peel_app(g, h)
        assert (g.stats()["k4_tail_launches"] > 0) == (engine == "1")
        g.free()
    want = got["0", None]
    for k in (("1", None), ("1", "0")):
        np.testing.assert_array_equal(got[k][0], want[0])
        assert got[k][1:] == want[1:]
    mem, rho, steps, best = oracle.Graph(*made).peel_app(h, rounds=True)
    np.testing.assert_array_equal(want[0].astype(bool), np.asarray(mem).astype(bool))
    assert want[1:] == (rho, steps, best)
