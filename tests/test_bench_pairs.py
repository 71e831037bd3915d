"""bench.py's roofline of a restore whose lattice search went by pairs: pairs and
the records they read, not addresses that the search never made."""
import bench


def test_a_search_by_pairs():
    t = {"hot_scan_ms": 0.01, "rows_ms": 0.02, "join_ms": 0.05, "estimate_ms": 0.01,
         "sort_publish_ms": 0.01, "hot_scan_bytes": 8e7, "join_probes": 0, "join_outputs": 5000,
         "estimate_bytes": 6.4e6, "search": 2, "lattice_points": 2e8, "pairs": 2_500_000}
    cs = bench.restore_roofline([t, t, t])["candidate_search"]
    assert cs["kind"] == "pairs" and cs["pairs"] == 2_500_000 and cs["outputs"] == 5000
    assert "points_per_s" not in cs and "frac" not in cs
    assert cs["pairs_per_s"] == 5e10
    assert abs(cs["achieved"] - bench.PAIR_RECORD_BYTES * 5e10 / 1e12) < 1e-3
    cs = bench.restore_roofline([dict(t, pairs=0)])["candidate_search"]
    assert cs["kind"] == "lattice" and cs["points"] == 2e8
