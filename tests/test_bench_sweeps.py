"""The roofline numerator that the benchmark reports for the propagation
sweeps, pinned for its pair (1024x436, k = 3, F and B1 with r = 8, B2 with 6):
one launch per sweep, four sweeps on each of four levels, nothing but sweeps in
them."""
import bench


def test_ops_per_sweep_launch():
    assert bench.sweep_launches_per_field(bench.K) == 16
    radii = (bench.R, bench.R, bench.R2)
    assert radii == (8, 8, 6)
    # 593,024 grid points over the levels; per point, two candidates of
    # 2 (2r + 1) terms, two operations each
    want = sum(593_024 * 4 * 2 * 2 * (2 * r + 1) * 2 for r in radii) / 48
    assert int(want) == 18_581_418
    assert bench.sweep_ops_per_launch(1024, 436, bench.K, radii) == want
