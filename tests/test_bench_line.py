"""What the benchmark's line says of its dominant launch, from the committed counter summaries (no GPU)."""
import json
import os

import pytest

PROFILES = os.path.join(os.path.dirname(os.path.abspath(__file__)), "..", "profiles")


@pytest.mark.parametrize("config,want", [(1, (0, "both")), (2, (0, "both")), (3, (0, "vms")), (5, (1, "vms")), (6, (0, "both"))])
def test_dominant_launch_has_its_recorded_counters(config, want):
    import bench
    lines = open(os.path.join(PROFILES, "replay_kernels_config%d_counters.txt" % config)).read().splitlines()
    counters = json.loads([l for l in lines if l.startswith("counters_json:")][0].split(":", 1)[1])
    # side by side in a run: a batch in one launch reports the same time for both policies
    batches = sorted({k.split("_")[0] for k in counters})
    per_batch = [dict(vms=9.0, split=9.0 if b + "_both" in counters else 8.0, total=9.5) for b in batches]
    b, p, ms, c = bench.dominant_launch(per_batch, counters)
    assert (b, p) == want and ms == 9.0
    assert c["hbm_bytes"] > 0 and c["lds"]["bytes"] > 0 and c["issue_rate"] and p in bench.BYTES_PER_EVENT and p in bench.POLICY_OF_LAUNCH


def test_dominant_launch_without_counters_is_the_longest():
    import bench
    b, p, ms, c = bench.dominant_launch([dict(vms=5.0, split=5.0), dict(vms=4.0, split=7.0)], {})
    assert (b, p, ms, c) == (1, "split", 7.0, {})
