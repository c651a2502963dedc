"""The shorter tiles a small plan takes when it is stepped alone."""
import numpy as np
import pytest

from paper_0802_3775_amd import workloads as W

pytestmark = pytest.mark.gpu


# a bound on the workgroups keeps the tuning's tiles: the same values from both,
# with energy samples (recorded by the tuning's tiles) every step, every third, in
# the last step only and never; energy sums group the same partial sums by other
# workgroup counts, so they are the same bit for bit too
@pytest.mark.parametrize("ke", [0, 1, 3, 22])
@pytest.mark.parametrize("kind", ["slab", "lorentz"])
def test_short_tiles_equal_tuned_tiles(kind, ke):
    import torch
    from paper_0802_3775_amd import fdtd
    steps = 23
    if kind == "slab":
        cfg = W.slab(res=9, cells=(3, 2, 2), steps=steps, nf=4, decim=3, energy_interval=ke)
    else:
        cfg = W.lasing(res=8, cells=(2, 2, 2), pml=5, steps=steps, noise=1e-3, energy_interval=ke)
    cfg["init_fields"] = {c: 1e-2 * a for c, a in W.random_fields(cfg["grid"]["n"], 3).items()}
    got = []
    for blocks in (0, 100000):
        plan = fdtd.Plan(cfg, max_steps=steps, tuning={"zchunk": 8, "graph_steps": 7, "max_blocks": blocks})
        plan.step(steps)
        torch.cuda.synchronize()
        out = [plan.fields(), plan.probe(0)]
        if plan.nf:
            out += list(plan.flux(0)) + list(plan.flux(1))
        if ke:
            out.append(plan.energy())
        if kind == "lorentz":
            out += [plan.populations(), plan.polarization()]
        got.append(out)
        plan.close()
    for a, b in zip(*got):
        assert np.array_equal(a, b)
