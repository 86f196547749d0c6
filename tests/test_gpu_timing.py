"""The times of the last call are a query: it disturbs no capture under way, and
waits for no work that other streams, the default one among them, have queued."""
import numpy as np
import pytest
import torch

from paper_2202_05012_amd import supa, workloads

pytestmark = pytest.mark.gpu


def timed_call(**how):
    w = workloads.WORKLOADS["e10_normal_5planes_1k"]
    sim = supa.Simulator(workloads.geometry(w), supa.OUT_HITS)
    sim.set_schedule(how.get("subs", 1), 0)
    ic = [torch.from_numpy(np.ascontiguousarray(a, np.float32)).cuda() for a in workloads.initial_conditions(w, 500)]
    out = sim.allocate(500, 1 << 18)
    assert sim.run(*ic, 3, out) == 0
    return sim


@pytest.mark.parametrize("subs", [1, 2])
def test_query_during_a_capture(subs):
    sim = timed_call(subs=subs)
    x, g = torch.zeros(8, device="cuda"), torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(g):
        y = x + 1
        ms = sim.timing()
        z = y * 2
    print(f"times during a capture: {ms}", flush=True)
    assert ms[2] >= ms[0] > 0 and ms[3] > 0
    assert ms == sim.timing()
    for rep in range(3):
        x.fill_(rep)
        g.replay()
        torch.cuda.synchronize()
        assert bool((z == 2 * (rep + 1)).all())


@pytest.mark.parametrize("side", [False, True])
def test_query_beside_queued_work(side):
    sim = timed_call()
    a = torch.rand(8192, 8192, device="cuda")
    b = a @ a
    torch.cuda.synchronize()
    with torch.cuda.stream(torch.cuda.Stream() if side else torch.cuda.current_stream()):
        for _ in range(60):
            torch.mm(a, a, out=b)
        done = torch.cuda.Event()
        done.record()
        ms = sim.timing()
        waited = done.query()
    torch.cuda.synchronize()
    assert ms[2] >= ms[0] > 0 and not waited
