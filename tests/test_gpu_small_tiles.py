"""DFT samples of tiles of few threads, which hold them among their staged fields."""
import numpy as np
import pytest

from gpu_common import rel_l2
from paper_0802_3775_amd import workloads as W

pytestmark = pytest.mark.gpu


# 64 threads hold the samples of up to three flux planes of a tile there, 128 of one,
# more and larger tiles elsewhere; planes of one tile, neighbouring and apart, sampled
# at different steps.  The same values as from tiles of 256 threads bit for bit (a tile's
# T(t) partial has another size, so T(t) to FP64 rounding); those tiles' spectra are
# compared with the FP64 reference where the device sums are tested.
@pytest.mark.parametrize("planes", [[(9, 1)], [(9, 1), (10, 2)], [(8, 1), (9, 1), (11, 3)],
                                    [(8, 2), (9, 1), (10, 1), (11, 1)]])
@pytest.mark.parametrize("block", [64, 128, 192])
def test_samples_of_small_tiles(block, planes):
    import torch
    from paper_0802_3775_amd import fdtd
    steps = 33
    cfg = W.homogeneous_box((37, 22, 24), (1, 1, 0), pml=(0, 0, 5), steps=steps)
    cfg["sources"] = [{"kind": "plane", "comp": 1, "k": 8, "f0": 0.8, "width_kind": "sigma_t", "width": 0.5,
                       "delay": 0.2, "amp": 1.0}]
    cfg["flux"] = [{"k": k, "freqs": (0.6, 0.75, 0.9), "decim": d} for k, d in planes]
    got = []
    for b in (block, 256):
        plan = fdtd.Plan(cfg, max_steps=steps, tuning={"tile_x": 16, "block": b, "zchunk": 8, "graph_steps": 8})
        plan.step(steps)
        torch.cuda.synchronize()
        got.append((plan.fields(), [plan.flux(f) for f in range(len(planes))]))
        plan.close()
    assert np.array_equal(got[0][0], got[1][0])
    for f in range(len(planes)):
        (t, s), (t1, s1) = got[0][1][f], got[1][1][f]
        assert np.array_equal(s, s1)
        assert rel_l2(t, t1) <= 1e-13
