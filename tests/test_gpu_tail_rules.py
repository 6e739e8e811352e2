"""Where the clique tail takes over, and which rounds its workgroup keeps, by
the counts it reports; results against closed forms and the round kernels."""
from math import comb

import numpy as np
import pytest

from paper_1906_00341_amd import dsd, synth
from test_gpu_clique_tail import _cliques, _dense

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


def test_six_clique_rounds_go_to_the_grid(monkeypatch):
    # single vertices of 50 to 150 members leave round after round: their
    # 5-cliques are a walk over the common neighbours of every triangle, more
    # than the workgroup keeps
    n, s, d = synth.rmat(scale=13, edge_factor=16, seed=5)
    got = {}
    for engine in ("1", "0"):
        monkeypatch.setenv("DSD_TAIL_ENGINE", engine)
        g = dsd.build_csr(n, s, d)
        core, km = dsd.clique_core(g, 6)
        got[engine] = core, km, g.stats()
        g.free()
    np.testing.assert_array_equal(got["1"][0], got["0"][0])
    assert got["1"][1] == got["0"][1]
    st = got["1"][2]
    assert st["k4_tail_launches"] > 0
    assert st["k4_tail_grid_pairs"] > st["k4_tail_pairs"]


def test_matrix_rebuilds_take_no_more_memory(monkeypatch):
    # 60,060 vertices in cliques of 5 to 60: the matrix is rebuilt four times on the way
    torch = pytest.importorskip("torch")
    dsd.load()
    n, s, d = _cliques(list(range(5, 61)) * 33)
    used = {}
    for engine in ("0", "1"):
        monkeypatch.setenv("DSD_TAIL_ENGINE", engine)
        dsd.release_cache()
        before = torch.cuda.mem_get_info()[0]
        g = dsd.build_csr(n, s, d)
        _, km = dsd.clique_core(g, 4)
        st = g.stats()
        g.free()                                     # (its memory stays for the next handle)
        used[engine] = before - torch.cuda.mem_get_info()[0]
        assert km == comb(59, 3)
    assert st["k4_tail_vertices"] > n                # rebuilt: some vertices count again
    words = n * -(-n // 64)
    need = 8 * 2 * words + 256 * n                   # the first matrix, one vertex's worst case beside it, lists
    assert used["1"] - used["0"] < need + (256 << 20)   # (memory comes in chunks of 64 MiB and more)


def test_batch_with_a_graph_above_the_tails_limit():
    # one graph of more than 131,072 vertices alive for nine rounds, where the
    # tail cannot take the batch; it takes the others' rounds after those
    sizes = list(range(5, 13)) * 20 + [13] * 10100
    made = [_cliques(sizes), _dense(200, 0.5, 3), _cliques(list(range(5, 41)))]
    alone = []
    for n, s, d in made[1:]:
        g = dsd.build_csr(n, s, d)
        alone.append(dsd.clique_core(g, 4))
        g.free()
    gs = [dsd.build_csr(*m) for m in made]
    outs = [np.zeros(m[0], np.uint64) for m in made]
    res = dsd.batch_run(gs, 4, "core", outs=outs)
    dsd.clique_core(gs[1], 4)                        # kept by the batch: its peel's figures
    assert gs[1].stats()["k4_tail_launches"] > 0
    for g in gs:
        g.free()
    want = np.concatenate([np.full(m, comb(m - 1, 3), np.uint64) for m in sizes])
    np.testing.assert_array_equal(np.sort(outs[0]), np.sort(want))
    assert res[0]["kmax"] == comb(12, 3)
    for (core, km), out, r in zip(alone, outs[1:], res[1:]):
        np.testing.assert_array_equal(out, core)
        assert r["kmax"] == km
