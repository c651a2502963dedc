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


# T(t) and energy records read as they grow, from fewer partial sums than the device
# takes (24,576) to more, in whole groups of 16 samples and with a part, 640 and 96
# partials a sample: every read begins with the one before, bit for bit, as both ways
# add a sample's partials up in the same order.
@pytest.mark.parametrize("nx,ny", [(68, 62), (20, 23)])
def test_records_grow(nx, ny):
    from paper_0802_3775_amd import fdtd
    reads = [1, 15, 38, 39, 48, 49, 255, 256, 257, 310, 1030, 2048, 2049]
    cfg = W.homogeneous_box((nx, ny, 24), (1, 1, 0), pml=(0, 0, 5), steps=reads[-1])
    cfg["sources"] = [{"kind": "plane", "comp": 1, "k": 8, "f0": 0.8, "width_kind": "sigma_t", "width": 0.5,
                       "delay": 0.2, "amp": 1.0}]
    cfg["flux"] = [{"k": 12, "freqs": (), "decim": 1}]
    cfg["energy_interval"] = 1
    plan = fdtd.Plan(cfg, max_steps=reads[-1], tuning={"tile_x": 16, "block": 64, "zchunk": 3})
    prev, last = (np.zeros(0), np.zeros(0)), 0
    for n in reads:
        plan.step(n - last)
        got, last = (plan.flux(0)[0], plan.energy()), n
        for a, b in zip(prev, got):
            assert len(b) == n and np.array_equal(a, b[:len(a)])
        prev = got
    assert np.all(prev[1][100:] > 0) and np.any(prev[0] != 0)
    plan.close()
