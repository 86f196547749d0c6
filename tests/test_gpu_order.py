"""Work order and the first batches dealt out by it: every shower is taken
exactly once whatever the number of waves, batches and sub-batches, at the
sizes where the last row of showers ends, and the order itself holds at the
size where one block stops ordering.  Per-shower results do not depend on the
order: exact (integers), against the batch order."""
import numpy as np
import pytest
import torch

from paper_2202_05012_amd import supa, workloads

pytestmark = pytest.mark.gpu


def run(sim, ics, n):
    ics = [a[:n].contiguous() for a in ics]
    out = sim.simulate(*ics, 7)
    return out["counts"].clone(), out["ledger"].clone(), out["total_hits"], out["total_steps"]


def ics(n, kind):
    rng = np.random.default_rng(n)
    e = {"equal": np.full(n, 3.0), "wide": np.exp(rng.uniform(np.log(0.1), np.log(30), n)),
         "edge": np.where(rng.random(n) < 0.2, 0.0, rng.uniform(0, 2, n))}[kind]
    t = lambda a: torch.from_numpy(a.astype(np.float32)).cuda()
    return t(e), t(rng.uniform(0, 0.5, n)), t(rng.uniform(0, 6, n))


@pytest.mark.parametrize("kind", ["equal", "wide", "edge"])
@pytest.mark.parametrize("subs", [1, 2, 3])
def test_every_shower_is_taken_once(kind, subs):
    w = workloads.WORKLOADS["e10_normal_5planes_1k"]
    geom = workloads.geometry(w)
    sim = supa.Simulator(geom, supa.OUT_HITS)
    data = ics(3100, kind)
    for n in (1, 2, 255, 256, 257, 511, 512, 513, 515, 767, 768, 769, 771, 1023, 1024, 1025, 1027, 2049, 3100):
        print(f"order: {n} showers, {kind} energies, {subs} sub-batches", flush=True)
        sim.set_launch(1)                                   # 256 waves
        sim.set_schedule(subs, 0)
        a = run(sim, data, n)
        sim.set_schedule(subs, 1)
        for _ in range(2):
            b = run(sim, data, n)
            assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1]) and a[2:] == b[2:]


@pytest.mark.parametrize("n", [4097, 16384, 32767, 32768, 32769, 40000])
def test_automatic_order(n):
    """More showers than waves, twelve planes: ordered by default."""
    print(f"order: {n} showers, automatic", flush=True)
    w = workloads.WORKLOADS["e10_normal_5planes_1k"]
    geom = workloads.geometry(w, n_planes=12)
    data = ics(n, "wide")
    sim = supa.Simulator(geom, supa.OUT_HITS)
    auto = run(sim, data, n)
    sim.set_schedule(1, 0)
    plain = run(sim, data, n)
    assert torch.equal(auto[0], plain[0]) and torch.equal(auto[1], plain[1]) and auto[2:] == plain[2:]


def test_captured_call_orders_at_each_replay():
    """5,000 showers of twelve planes: the work order is part of the captured
    call and follows the energies the input holds at the replay."""
    w = workloads.WORKLOADS["e10_normal_5planes_1k"]
    geom = workloads.geometry(w, n_planes=12)
    n = 5000
    a, b = ics(n, "wide"), ics(n, "edge")
    sim = supa.Simulator(geom, supa.OUT_HITS)
    eager = [run(sim, d, n) for d in (a, b)]
    args = [t.clone() for t in a]
    out = sim.allocate(n, 1 << 22)
    assert sim.run(*args, 7, out) == 0
    g = sim.graph(*args, 7, out)
    for rep, d in enumerate((a, b, a)):
        print(f"order: replay {rep}", flush=True)
        for t, s in zip(args, d):
            t.copy_(s)
        out["counts"].fill_(-1)
        g.launch()
        g.check()
        torch.cuda.synchronize()
        ref = eager[rep % 2]
        assert torch.equal(out["counts"], ref[0]) and torch.equal(out["ledger"], ref[1])
        assert out["total_hits"] == ref[2]
    g.close()


def test_pipelined_calls_with_a_work_order():
    """Calls of 5,000, 4,097 and 6,000 showers, each ordered, in one entry."""
    print("order: three calls in one", flush=True)
    w = workloads.WORKLOADS["e10_normal_5planes_1k"]
    geom = workloads.geometry(w, n_planes=12)
    sizes = [5000, 4097, 6000]
    data = ics(sum(sizes), "wide")
    sim = supa.Simulator(geom, supa.OUT_HITS)
    calls = [(sum(sizes[:j]), m) for j, m in enumerate(sizes)]
    outs = [sim.allocate(m, 1 << 21) for m in sizes]
    assert sim.run_batches(*data, 7, calls, outs) == 0
    for (s0, m), o in zip(calls, outs):
        ref = sim.simulate(*[t[s0:s0 + m].contiguous() for t in data], 7, shower_id_base=s0)
        assert torch.equal(o["counts"], ref["counts"]) and torch.equal(o["ledger"], ref["ledger"])
        assert torch.equal(o["hit_offsets"], ref["hit_offsets"]) and o["total_hits"] == ref["total_hits"]


@pytest.mark.parametrize("sizes", [[0, 0], [0, 700, 0], [300, 0, 500, 0, 0, 40, 600]])
def test_pipelined_calls_some_of_them_empty(sizes):
    """Calls without showers between others: nothing to do, totals of zero."""
    print(f"order: calls of {sizes} showers in one", flush=True)
    w = workloads.WORKLOADS["e10_normal_5planes_1k"]
    sim = supa.Simulator(workloads.geometry(w), supa.OUT_HITS)
    data = ics(max(1, sum(sizes)), "wide")
    calls = [(sum(sizes[:j]), m) for j, m in enumerate(sizes)]
    outs = [sim.allocate(m, 1 << 18) for m in sizes]
    for _ in range(2):
        assert sim.run_batches(*data, 7, calls, outs) == 0
        for (s0, m), o in zip(calls, outs):
            ref = sim.simulate(*[t[s0:s0 + m].contiguous() for t in data], 7, shower_id_base=s0)
            assert torch.equal(o["counts"], ref["counts"]) and torch.equal(o["ledger"], ref["ledger"])
            assert all(o[k] == ref[k] for k in ("total_hits", "total_nodes", "total_steps"))
            assert m > 0 or o["total_steps"] == 0


def by_key(o, pre, col, fields):
    """A call's records in the order of showers and path ids (segments follow one another)."""
    c = o["counts"][:, col].long()
    shower = torch.repeat_interleave(torch.arange(c.numel(), device=c.device), c)
    m = shower.numel()
    i = o[pre + "_key"][:m].argsort()
    i = i[shower[i].argsort(stable=True)]
    return [o[f"{pre}_{f}"][:m][i] for f in fields]


# subtree items, orders of both kinds and no order in one entry, either way round
@pytest.mark.parametrize("sizes", [[200, 40000, 4097, 3000, 33000, 100], [4097, 200, 5000, 40000, 3000]])
def test_pipelined_calls_of_every_kind_share_one_layout(sizes):
    print(f"order: calls of {sizes} showers in one, every output", flush=True)
    w = workloads.WORKLOADS["e10_normal_5planes_1k"]
    geom = workloads.geometry(w, n_planes=12, img_nx=8, img_ny=8, img_x0=-4.0, img_x1=4.0,
                              img_y0=-4.0, img_y1=4.0)
    data = ics(sum(sizes), "wide")
    sim = supa.Simulator(geom, supa.OUT_HITS | supa.OUT_KEYS | supa.OUT_TREE | supa.OUT_IMAGES)
    calls = [(sum(sizes[:j]), m) for j, m in enumerate(sizes)]
    alone = [sim.simulate(*[t[s0:s0 + m].contiguous() for t in data], 7, shower_id_base=s0) for s0, m in calls]
    outs = [sim.allocate(m, r["total_hits"], r["total_nodes"]) for (_, m), r in zip(calls, alone)]
    for _ in range(2):
        for o in outs:
            o["images"].fill_(-1.0)
            o["hit_key"].zero_()
            o["node_key"].zero_()
        assert sim.run_batches(*data, 7, calls, outs) == 0
        for o, r in zip(outs, alone):
            for k in ("counts", "ledger", "hit_offsets", "node_offsets", "images"):
                assert torch.equal(o[k], r[k]), k
            for a, b in zip(by_key(o, "hit", 1, ("x", "y", "e", "layer", "key")) +
                            by_key(o, "node", 0, ("gen", "vx", "vy", "vz", "e", "key")),
                            by_key(r, "hit", 1, ("x", "y", "e", "layer", "key")) +
                            by_key(r, "node", 0, ("gen", "vx", "vy", "vz", "e", "key"))):
                assert torch.equal(a, b)
