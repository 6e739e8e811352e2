"""Min cuts on the GPU against the host's, on networks whose searches have wide
levels (pulled from the unlabelled nodes) and narrow ones (pushed from the
frontier), with vertex nodes below and above 4,096 arcs.  The densest subgraph's
members and density: equality."""
import numpy as np
import pytest

from paper_1906_00341_amd import dsd, synth

pytestmark = pytest.mark.gpu

CASES = {
    # (made, h)
    "dense, every vertex node large": (lambda: synth.chung_lu(n=400, avg_deg=150.0, beta=3.0, planted=1, plant_size=190,
                                                             p=0.9, seed=3), 3),
    "vertex nodes on both sides of 4,096 arcs": (lambda: synth.chung_lu(n=900, avg_deg=60.0, beta=2.2, planted=2,
                                                                        plant_size=110, p=0.8, seed=4), 3),
    "small": (lambda: synth.chung_lu(n=300, avg_deg=8.0, beta=2.3, planted=2, plant_size=20, p=0.7, seed=5), 3),
    "edges": (lambda: synth.chung_lu(n=5000, avg_deg=12.0, beta=2.3, planted=2, plant_size=60, p=0.5, seed=6), 2),
    "four-cliques": (lambda: synth.chung_lu(n=500, avg_deg=20.0, beta=2.3, planted=2, plant_size=40, p=0.7, seed=7), 4),
}


@pytest.mark.parametrize("name", list(CASES))
def test_gpu_cut_matches_host_cut(monkeypatch, name):
    make, h = CASES[name]
    made = make()
    got = {}
    for arcs in ("0", "-1"):
        monkeypatch.setenv("DSD_FLOW_GPU_MIN_ARCS", arcs)
        g = dsd.build_csr(*made)
        member, rho = dsd.core_exact(g, h)
        st = g.stats()
        g.free()
        assert st["flow_gpu_calls"] == (st["flow_calls"] if arcs == "0" else 0)
        got[arcs] = (np.asarray(member).copy(), rho)
    assert got["0"][1] == got["-1"][1]
    np.testing.assert_array_equal(got["0"][0], got["-1"][0])
