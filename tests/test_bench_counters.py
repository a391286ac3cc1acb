"""The counter summary behind the bench line's bytes per stage: launches counted
per step, and template arguments left aside when a stage's kernels are looked up."""
import os

import bench

# launches that a step of 2,097,152 particles makes by construction (three
# digit passes, their first histogram taken while the keys are computed)
PER_STEP = {"k_keys_hist": 1, "k_hist": 2, "k_digit_scan": 3, "k_scatter": 3, "k_local_sort": 1, "k_pack4": 1,
            "k_gather4": 1, "k_cluster_bbox": 1, "k_leaf_level": 1, "k_node_range": 1, "k_traverse": 1, "k_encode": 1,
            "k_pass_half": 1, "k_pass_finalize": 1}


def test_committed_summary_counts_launches_per_step():
    seen = {}
    with open(os.path.join(bench.ROOT, "profiles", "counters_uniform_2m.txt")) as f:
        for line in f:
            if line.startswith("traffic "):
                kv = dict(t.split("=", 1) for t in line.split()[1:])
                seen[kv["kernel"].split("<")[0]] = float(kv["launches_per_step"])
    assert {k: seen[k] for k in PER_STEP} == PER_STEP


def test_stage_bytes_take_every_kernel_of_the_stage():
    counters = {"k_leaf_level<4>": (3.0, 1.0), "k_emit_nodes<false>": (5.0, 1.0), "k_node_range<2>": (7.0, 1.0),
                "k_children": (11.0, 1.0), "k_box_levels": (13.0, 2.0), "k_node_slots": (17.0, 1.0),
                "k_cluster_bbox<8,true>": (19.0, 1.0), "k_pack4": (23.0, 1.0)}
    assert bench.stage_counter_bytes("octree", counters) == 3 + 5 + 7 + 11 + 26 + 17
    assert bench.stage_counter_bytes("clusters", counters) == 19
    assert bench.stage_counter_bytes("gather", counters) is None  # k_gather4 not measured
    assert bench.stage_counter_bytes("pass", counters) is None
