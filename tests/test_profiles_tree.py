"""The prefix-shared forward's committed counter summary belongs to the present
kernel source, so that the benchmark reports its traffic and not a null."""
import os
import re
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_tree_traffic_summary_is_current():
    sys.path.insert(0, ROOT)
    import bench
    text = open(os.path.join(ROOT, "profiles", "tree_forward_c4_bf16w_traffic.md")).read()
    m = re.search(r"kernel_source_sha256:\s*`?([0-9a-f]{64})", text)
    assert m and m.group(1) == bench.kernel_source_hash("tree_forward"), "counter summary taken on another source"
    # the states make it thousands of bytes per row, where row by row there are 24
    assert bench.tree_traffic("c4", "bf16w") > 1000.0
