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
