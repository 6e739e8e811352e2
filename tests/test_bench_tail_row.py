"""bench.py's roofline row of the clique tail: timed and counted as a whole, so
named after all of its kernels and without the traffic of any one of them."""
from __future__ import annotations

import bench


def test_clique_tail_row():
    st = {"k4_main_kind": 6, "k4_tail_pairs": 1000, "k4_tail_grid_pairs": 500, "k4_tail_vertices": 10}
    assert bench.tail_kernel_bytes(st) == 4 * 1500 + 20 * 10
    for kernel in ("k_ct_engine", "k_ct_front", "k_ct_edges", "k_ct_count"):
        assert kernel in bench.CLIQUE_TAIL
    r = bench.roof(bench.CLIQUE_TAIL, "rmat22_h4", 10.0, 5, bench.tail_kernel_bytes(st))
    assert r["ms_per_launch"] == 2.0 and r["traffic"] is None
