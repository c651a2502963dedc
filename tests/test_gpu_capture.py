"""Steps captured into the caller's own graph: the spectra after replays at any phase of
the DFT rings, and of eager steps while captured ones wait to be replayed."""
import numpy as np
import pytest

from paper_0802_3775_amd import workloads as W

pytestmark = pytest.mark.gpu

RING = 32  # samples per DFT launch
STEPS = 24 + 8 * 40  # past three rings of decim 3, replays of 8 steps


def _cfg(decims, seed=3):
    c = W.slab(res=8, cells=(2, 2, 1), steps=STEPS, nf=9, decim=1, energy_interval=10, seed=seed)
    c["flux"] = [dict(f, decim=d) for f, d in zip(c["flux"], decims)]
    c["init_fields"] = W.random_fields(c["grid"]["n"], 4)
    return c


def _graph(step, n, stream):
    import torch
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=stream):
        step(n, stream=stream)
    return g


def _compare(plans, want):
    for p, w in zip(plans, want):
        assert p.step_count == w.step_count
        assert np.array_equal(p.fields(), w.fields())
        for f in range(len(w.nf)):
            for a, b in zip(p.flux(f), w.flux(f)):
                assert np.array_equal(a, b)


# A graph of 8 steps replayed again and again: with decim 3 and 5 its replays come to a
# full ring at offsets of the graph that held no sample when it was captured.  A capture
# counts its steps on the host, so one capture is made per replay.
@pytest.mark.parametrize("decims", [(3, 3), (5, 1), (8, 2)])
@pytest.mark.parametrize("batch", [False, True])
def test_replayed_graph_spectra(decims, batch):
    import torch
    from paper_0802_3775_amd import fdtd
    cfgs = [_cfg(decims), _cfg(decims[::-1], seed=5)] if batch else [_cfg(decims)]
    want = [fdtd.Plan(c, max_steps=STEPS) for c in cfgs]
    plans = [fdtd.Plan(c, max_steps=STEPS) for c in cfgs]
    st = fdtd.Batch(plans) if batch else plans[0]
    s = torch.cuda.Stream()
    st.step(3, stream=s)  # out of step with the rings
    s.synchronize()
    graphs = [_graph(st.step, 8, s) for _ in range(40)]
    for q in range(40):
        graphs[0].replay()
        if q % 13 == 0:
            torch.cuda.synchronize()
    torch.cuda.synchronize()
    st.step(STEPS - 3 - 320, stream=s)  # eager again
    s.synchronize()
    for w in want:
        w.step(STEPS)
    _compare(plans, want)
    del graphs
    if batch:
        st.close()
    for p in plans + want:
        p.close()


# eager steps between a capture and its replay: the device is behind the host's count
def test_eager_steps_before_replay():
    import torch
    from paper_0802_3775_amd import fdtd
    cfg = _cfg((1, 1))
    want, plan = fdtd.Plan(cfg, max_steps=STEPS), fdtd.Plan(cfg, max_steps=STEPS)
    s = torch.cuda.Stream()
    plan.step(5, stream=s)
    s.synchronize()
    g = _graph(plan.step, 7, s)
    plan.step(3 * RING, stream=s)
    s.synchronize()
    g.replay()
    torch.cuda.synchronize()
    plan.step(41, stream=s)
    s.synchronize()
    want.step(5 + 7 + 3 * RING + 41)
    _compare([plan], [want])
    del g
    plan.close()
    want.close()
