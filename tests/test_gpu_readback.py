"""Copies between the dense host arrays and the device's rows (padded or not)."""
import numpy as np
import pytest

from paper_0802_3775_amd import workloads as W

pytestmark = pytest.mark.gpu


# rows of 64 and 37 cells are not padded, rows of 60 and 250 are (64, 256); the
# copies of padded rows move in 2 MiB pieces, here less than one (60 x 7 x 5),
# one and a part (60 x 60 x 160) and several with a short last one (250 x 41 x 130)
@pytest.mark.parametrize("n", [(64, 9, 5), (37, 11, 6), (60, 7, 5), (60, 60, 160), (250, 41, 130), (1, 1, 33)])
def test_fields_and_map_round_trip(n):
    from paper_0802_3775_amd import fdtd
    cfg = W.homogeneous_box(n, materials=[{"eps": 1.0}, {"eps": 2.0}, {"eps": 3.0}], steps=1)
    cfg["map"] = W.random_map(n, 3, 5)
    plan = fdtd.Plan(cfg, max_steps=1)
    assert np.array_equal(plan.material_map(), cfg["map"])
    f = {c: np.float32(a) for c, a in W.random_fields(n, 8).items()}
    for c, a in f.items():
        plan.write_field(c, a)
    for c, a in f.items():
        assert np.array_equal(plan.field(c), a)
    plan.close()


# the device sums of a read: spectrum parts of 4,096 plane points (one short part,
# one whole, two with a short second; padded rows at 60 cells) and T(t) / energy
# samples in groups of 16 rows and 128 columns (15, 16, 17 and 33 samples; 80 to
# 700 partial sums each).  FP32 steps are within 33 * 6e-8 of the FP64 oracle's
# fields and products of two of them within twice that: 4e-6; the sums' cells agree
# in sign, so the bar is 1e-5.
@pytest.mark.parametrize("nx,ny,steps", [(20, 20, 15), (64, 64, 16), (68, 62, 17), (60, 70, 33)])
def test_flux_and_energy_sums(nx, ny, steps):
    from gpu_common import rel_l2, run_gpu, run_oracle
    cfg = W.homogeneous_box((nx, ny, 24), (1, 1, 0), pml=(0, 0, 5), steps=steps)
    cfg["sources"] = [{"kind": "plane", "comp": 1, "k": 8, "f0": 0.8, "width_kind": "sigma_t", "width": 0.5,
                       "delay": 0.2, "amp": 1.0}]
    cfg["flux"] = [{"k": 12, "freqs": (0.6, 0.75, 0.9), "decim": 1}]
    cfg["energy_interval"] = 1
    plan = run_gpu(cfg, steps, tuning={"tile_x": 16, "block": 64, "zchunk": 3, "graph_steps": 0})
    ref = run_oracle(cfg, steps)
    (T, S), (T0, S0) = plan.flux(0), ref.flux(0)
    assert len(T) == steps and rel_l2(T, T0) <= 1e-5 and rel_l2(S, S0) <= 1e-5
    W1, W0 = plan.energy(), ref.energy()
    assert len(W1) == len(W0) and rel_l2(W1, W0) <= 1e-5
    plan.close()
