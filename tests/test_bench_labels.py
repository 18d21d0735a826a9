"""The kernel names of the benchmark's step legs, on the CPU."""
import json

import pytest

import bench


@pytest.mark.parametrize("storage,file", [("fp32", "step2_f32"), ("fp16", "step_f16"), ("bf16", "step_bf16")])
def test_kernel_is_named_where_a_profile_saw_it(storage, file):
    """With a profile of the lattice: its kernel and steps per launch; on any
    other lattice no kernel is named."""
    with open(bench.PROFILE_TRAFFIC[file]) as fh:
        t = json.load(fh)
    label = bench.kernel_label(storage, False, t["n_nodes"])
    if t["kernel_sha"] == bench.kernel_source_hash():
        assert label.split("<")[0] in t["kernel"]
        assert label.endswith("two steps per launch" if t["updates_per_node"] == 2 else "one step per launch")
    else:
        assert "_kernel" not in label
    for n in (64, 1024):
        assert "_kernel" not in bench.kernel_label(storage, False, n * n)
    assert bench.kernel_label(storage, True, 64 * 64) == f"step_kernel<{storage.upper()}>, one step per launch"
