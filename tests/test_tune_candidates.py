"""The tuner's candidates run with the z-chunk that they name."""
import pytest

from paper_0802_3775_amd import fdtd, tune
from paper_0802_3775_amd import workloads as W


# A small plan stepped alone lays out shorter tiles of its own beside the tuning's (its
# arena holds both tables) unless its workgroups are bounded; with them several
# candidates are the same launch, and the chunk kept among them is noise.
@pytest.mark.parametrize("cfg", [W.periodic_cell(res=32, steps=8), W.slab(res=16, cells=(4, 4, 4), steps=8),
                                 W.lasing(res=12, cells=(4, 4, 4), steps=8)])
def test_candidates_keep_their_chunk(cfg):
    def arena(t, **kw):
        plan = fdtd.Plan(cfg, max_steps=8, tuning=dict(t, graph_steps=0, **kw), bind=False)
        try:
            return plan.required_bytes()
        finally:
            plan.close()

    cands = tune.candidates(cfg)
    assert {c["zchunk"] for c in cands} >= {1, 2, 4, 8, 16, 32}
    assert any(arena(c, max_blocks=0) != arena(c, max_blocks=7) for c in cands)  # a small plan
    for c in cands:
        assert arena(c) == arena(c, max_blocks=7)
