"""What bench.py divides by the stages' times: only bytes that a stage's kernels move."""
import pytest

import bench
from workloads import WORKLOADS


@pytest.mark.parametrize("name,k,stages", [("tiny", 1, {"gate"}), ("tiny", 2, {"gate", "combine"}), ("skew", 1, {"gate"}), ("large", 2, {"gate", "combine"})])
def test_stages_with_a_bandwidth(name, k, stages):
    wl = WORKLOADS[name].scaled(k=k)
    R = k * wl.T
    b = bench.hbm_stage_bytes(wl, R)
    assert set(b) == stages
    size = 4 if wl.dtype == "f32" else 2
    assert b["gate"] == wl.T * (wl.d_model * size + 8 * k)
    if "combine" in b:
        assert b["combine"] == (R + wl.T) * wl.d_model * size + 8 * k * wl.T
