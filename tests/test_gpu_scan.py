"""Segment offsets: one block scans up to 16,384 showers (64 * ceil(n / 1024)
consecutive ones per wave), three kernels scan more.  Offsets, totals and the
counters that the scan hands to the host, at the sizes where a wave's share
ends, for hits, nodes and both, in one and in several sub-batches.  Integers:
exact."""
import numpy as np
import pytest
import torch

from paper_2202_05012_amd import supa, workloads

pytestmark = pytest.mark.gpu

HT = supa.OUT_HITS | supa.OUT_TREE


@pytest.mark.parametrize("n", [1, 63, 65, 1023, 1024, 1025, 4097, 16383, 16384, 16385])
@pytest.mark.parametrize("outputs,subs", [(supa.OUT_HITS, 1), (supa.OUT_TREE, 1), (HT, 1), (HT, 3), (0, 1)])
def test_offsets_are_the_prefix_sums(n, outputs, subs):
    print(f"scan: {n} showers, outputs {outputs}, {subs} sub-batches", flush=True)
    w = workloads.WORKLOADS["e10_normal_5planes_1k"]
    geom = workloads.geometry(w)
    rng = np.random.default_rng(n)
    t = lambda a: torch.from_numpy(a.astype(np.float32)).cuda()
    ics = t(rng.uniform(0.5, 30, n)), t(rng.uniform(0, 0.3, n)), t(rng.uniform(0, 6, n))
    sim = supa.Simulator(geom, outputs)
    if subs > 1:
        sim.set_schedule(subs, 0)
    for seed in (1, 2):
        out = sim.simulate(*ics, seed)
        c = out["counts"].view(-1, 6).to(torch.int64)
        steps = out["total_steps"]
        assert steps > 0
        for flag, off, col, total in ((supa.OUT_HITS, "hit_offsets", 1, "total_hits"),
                                      (supa.OUT_TREE, "node_offsets", 0, "total_nodes")):
            if not outputs & flag:
                assert out[total] == 0
                continue
            assert torch.equal(out[off], c[:, col].cumsum(0) - c[:, col])
            assert out[total] == int(c[:, col].sum())
        ms = sim.timing()
        assert ms[2] >= ms[0] > 0 and min(ms) >= 0, ms
