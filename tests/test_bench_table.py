"""The stage table of bench.py counts the launches of each stage."""
import bench


def test_launches_of_the_depth_first_frame():
    st = dict(N=1_000_000, V=700_000, K=1_500_000, S=1000, passes=2, dpasses=2, tiles=2040, pix=1920 * 1080, evals=1, keff=1)
    bytes_, flops = bench.algorithmic_model(st, 4, 3)
    stages = dict(preprocess=0.05, scan=0.02, readback=0.0, depth_sort=0.03, emit=0.03, key_sort=0.03, ranges=0.005, blend=0.1)
    table, launches = bench.stage_table(stages, bytes_, flops, st)
    assert bench.SORT_MODE == 0
    # reduce, row scan, down; the same per depth pass; reduce, offsets, down; the first key pass without its count
    assert launches == {"scan": 3, "depth_sort": 6, "emit": 3, "key_sort": 5}
    assert table["emit"]["launches"] == 3 and table["emit"]["avg_launch_ms"] == 0.01
    assert bench.stage_table(stages, bytes_, flops, dict(st, V=3_000_000))[1]["emit"] == 4   # the sums scanned by a launch of their own
