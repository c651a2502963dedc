"""Records longer than one pass of the device sums' workgroups."""
import numpy as np
import pytest

from paper_0802_3775_amd import workloads as W

pytestmark = pytest.mark.gpu


# 65,536 samples are one row per thread of all workgroups of the sums; the rest takes a
# second turn.  The energy of a lossless periodic box is constant to the FP32 rounding
# of the fields (6e-8 a step, 4e-3 over all steps if every error had one sign); a sample
# that was not summed is 0.
def test_energy_beyond_one_pass():
    from paper_0802_3775_amd import fdtd
    steps = 65536 + 1003
    cfg = W.homogeneous_box((8, 8, 8), steps=steps)
    cfg["init_fields"] = W.random_fields((8, 8, 8), 6)
    cfg["energy_interval"] = 1
    plan = fdtd.Plan(cfg, max_steps=steps, tuning={"tile_x": 16, "block": 64})
    plan.step(steps)
    w = plan.energy()
    assert len(w) == steps and w[0] > 0
    assert np.max(np.abs(w / w[0] - 1.0)) <= 1e-2
    plan.close()
