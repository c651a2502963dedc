"""Boxes with CPML on all axes: tiles off the x and y slabs in the all-axes launch."""
import numpy as np
import pytest

from gpu_common import field_rel_l2, pec_clean, rel_l2, run_oracle
from paper_0802_3775_amd import workloads as W

pytestmark = pytest.mark.gpu


def _cfg(nx, steps):
    # one full 64-cell tile column between the x slabs; tiles with z-slab planes
    # only, none and all; sources and probes in some
    n = (nx, 29, 23)
    cfg = W.homogeneous_box(n, (0, 0, 0), pml=(7, 5, 4), materials=[{"eps": 1.0}, {"eps": 2.5}], steps=steps)
    cfg["map"] = W.random_map(n, 2, 3)
    cfg["init_fields"] = {c: a.astype(np.float32) for c, a in pec_clean(
        W.random_fields(n, 8), cfg["grid"]["periodic"]).items()}
    cfg["sources"] = [{"kind": "dipole", "comp": 1, "i": 70, "j": 12, "k": 11, "f0": 0.8, "width_kind": "fwhm_power",
                       "width": 0.3, "delay": 0.1, "amp": 1.0}]
    cfg["probes"] = [(0, 80, 14, 20), (4, 100, 16, 9), (5, 2, 2, 2)]
    return cfg


# one launch of all classes (merge 2) and one per class (merge 0): each tile steps
# through the same arithmetic in both, so the same values bit for bit; against the
# FP64 reference the project's bound for FP32 fields
@pytest.mark.parametrize("tile_x", [16, 32, 64])
@pytest.mark.parametrize("nx", [143, 160])
def test_interior_march_of_all_axes_launch(nx, tile_x):
    import torch
    from paper_0802_3775_amd import fdtd
    steps = 24
    cfg = _cfg(nx, steps)
    got = []
    for merge in (0, 2):
        plan = fdtd.Plan(cfg, max_steps=steps, tuning={"tile_x": tile_x, "block": 256, "zchunk": 6, "merge": merge})
        plan.step(steps)
        torch.cuda.synchronize()
        got.append((plan.fields(), [plan.probe(q) for q in range(3)]))
        plan.close()
    assert np.array_equal(got[0][0], got[1][0])
    for a, b in zip(got[0][1], got[1][1]):
        assert np.array_equal(a, b)
    orc = run_oracle(cfg, steps)
    assert field_rel_l2(got[1][0], orc.fields()) <= 1e-4
    for q in range(3):
        assert rel_l2(got[1][1][q], orc.probe(q)) <= 1e-4
