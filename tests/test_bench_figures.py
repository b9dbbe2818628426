"""Figures that bench.py stores rather than measures, against the profiles they come from and against what they are per."""
import os
import re

import bench
from kvp_workload import chunk_ranges, get_workload

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_stored_attention_traffic_is_per_launch_of_as_many_layers():
    wl = get_workload("long_video")
    text = open(os.path.join(ROOT, "profiles", "long_video_prefill_hbm_traffic.txt")).read()
    layers = int(re.search(r"^LAYERS_PER_LAUNCH (\d+)$", text, re.M).group(1))
    stored = int(re.search(r"^TRAFFIC_BYTES (\d+)$", text, re.M).group(1))
    assert bench.attention_traffic("long_video", layers) == bench.attention_traffic("long_video", float(layers)) == stored
    assert bench.attention_traffic("long_video", 1) is None and bench.attention_traffic("video", layers) is None
    # every query, key and value in and every output out, once: the launch cannot move less, and moves the keys
    # again for the second sweep and the partial scores
    total, c, blocks = 0, 0, chunk_ranges(wl.n_tokens, wl.chunk)
    for _, n in blocks:
        total += wl.head_dim * 2 * (2 * n * wl.n_q_heads + 2 * (c + n) * wl.n_kv_heads) + 4 * n * wl.n_q_heads
        c = min(wl.budget, c + n)
    least = layers * total / len(blocks)
    assert least <= stored <= 3 * least
