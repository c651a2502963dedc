"""Density-matrix passes at the sizes and places where their indexing can go wrong."""
import numpy as np
import pytest

from gpu_common import field_rel_l2, rel_l2, run_oracle
from paper_0802_3775_amd import workloads as W

pytestmark = pytest.mark.gpu


# rows and planes below, at and beyond the 8-row blocks and the 32-cell padding, one
# cell thick axes, gain cells on PEC walls and across periodic ones; nine in ten
# cells have gain, so that the largest grid fills more than the 256 units that are
# dealt to the XCDs in runs.  The bar is the one of the other density-matrix
# checks against the oracle (FP32 rounding over a few dozen steps: 1e-4).
@pytest.mark.parametrize("n,per", [((1, 9, 8), (1, 1, 1)), ((7, 1, 17), (0, 1, 0)), ((33, 8, 9), (1, 0, 1)),
                                   ((30, 17, 16), (0, 0, 0)), ((64, 40, 33), (0, 1, 0))])
def test_passes_match_oracle_and_probes_match_fields(n, per):
    import torch
    from paper_0802_3775_amd import fdtd
    nx, ny, nz = n
    steps = 24
    cfg = W.homogeneous_box(n, per, materials=[{"eps": 2.0}, W.density_material(noise=1e-3)], steps=steps)
    cfg["map"] = (np.random.default_rng(2).random((nz, ny, nx)) < 0.9).astype(np.uint8)
    cfg["map"][nz // 2:, :, : (nx + 1) // 2] = 0  # and a part of the grid without any
    f = {c: 1e-2 * a for c, a in W.random_fields(n, 6).items()}
    cfg["init_fields"] = f
    # probes of every component in gain cells, beside them, far from them and on the walls
    cells = [(0, 0, 0), (nx - 1, ny - 1, nz - 1), (nx // 2, ny // 2, 0), (0, 0, nz - 1)]
    cfg["probes"] = [(c % 6,) + cells[q % 4] for q, c in enumerate(range(16))]
    plan = fdtd.Plan(cfg, max_steps=steps)
    for chunk in (1, 2, 21):
        plan.step(chunk)
        torch.cuda.synchronize()
        fields = plan.fields()
        for q, (c, i, j, k) in enumerate(cfg["probes"]):  # recorded after the edge pass
            assert plan.probe(q)[-1] == fields[c][k, j, i], (chunk, q)
    ref = run_oracle(cfg, steps)
    gain = cfg["map"] == 1
    assert field_rel_l2(plan.fields(), ref.fields()) <= 1e-4
    assert rel_l2(plan.density()[:, gain], ref.density()[:, gain]) <= 1e-4
    plan.close()
