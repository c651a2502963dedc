"""Step calls cut into runs at the DFT launches, with graphs of repeated lengths."""
import numpy as np
import pytest

from paper_0802_3775_amd import workloads as W

pytestmark = pytest.mark.gpu

CHUNKS = [3, 3, 25, 1, 32, 31, 33, 64, 7, 7, 7, 7, 7, 9, 9, 128, 2, 2, 2]  # ring ends at 31, 63, ...


def _cfgs(steps):
    a = W.slab(res=8, cells=(2, 2, 1), steps=steps, nf=9, decim=1, energy_interval=10)   # a ring of 32 steps
    a["flux"][1] = dict(a["flux"][1], decim=3)                                         # and one of 96
    b = W.slab(res=9, cells=(2, 1, 1), steps=steps + 50, nf=5, decim=2, energy_interval=7, seed=3)
    for c in (a, b):
        c["init_fields"] = W.random_fields(c["grid"]["n"], 4)
    return a, b


def _out(p):
    return [p.fields(), p.probe(0), p.energy()] + [v for f in range(2) for v in p.flux(f)]


@pytest.mark.parametrize("graph_steps", [1, 5, 64])
@pytest.mark.parametrize("batch", [False, True])
def test_runs_equal_eager(graph_steps, batch):
    import torch
    from paper_0802_3775_amd import fdtd
    steps = sum(CHUNKS)
    got = []
    for g in (0, graph_steps):
        plans = [fdtd.Plan(c, max_steps=c["steps"], tuning={"graph_steps": g}) for c in _cfgs(steps)]
        plans[1].step(45)  # members out of step: the second's rings end elsewhere
        st = fdtd.Batch(plans) if batch else plans[0]
        for c in CHUNKS if g else [steps]:
            st.step(c)
        torch.cuda.synchronize()
        got.append([_out(p) for p in plans])
        if batch:
            st.close()
        for p in plans:
            p.close()
    for a, b in zip(*got):
        for x, y in zip(a, b):
            assert np.array_equal(x, y)


# a graph captured by the caller, replayed to and past a full ring: every sample's
# DFT launch is in it, and the kernel looks at the step
def test_caller_captured_steps():
    import torch
    from paper_0802_3775_amd import fdtd
    cfg = _cfgs(80)[0]
    want = fdtd.Plan(cfg, max_steps=80)
    want.step(80)
    plan = fdtd.Plan(cfg, max_steps=80)
    s = torch.cuda.Stream()
    plan.step(8, stream=s)
    s.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=s):
        plan.step(8, stream=s)  # counted once here, run by the replays
    for _ in range(8):
        graph.replay()
    torch.cuda.synchronize()
    # the device has made 72 steps and the plan counts 16: step the last 8 by hand
    graph.replay()
    torch.cuda.synchronize()
    a, b = plan.fields(), want.fields()
    assert np.array_equal(a, b)
    del graph
    plan.close()
    want.close()
