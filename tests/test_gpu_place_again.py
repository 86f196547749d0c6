"""Arrays too small for a call's records: the records, still in the library's
logs, are placed again into larger ones.  Against the oracle (as a call with
enough room), for every kind of record, with items, sub-batches and a work
order; and the cases with nothing to place again."""
import ctypes as C

import numpy as np
import pytest
import torch

from oracle import supa_oracle as O
from paper_2202_05012_amd import supa, workloads
from tests import parity

pytestmark = pytest.mark.gpu

H, I, T, K = supa.OUT_HITS, supa.OUT_IMAGES, supa.OUT_TREE, supa.OUT_KEYS


def ics(w, n):
    e0, pol, az = workloads.initial_conditions(w, n)
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a, np.float32)).cuda()
    return (e0, pol, az), (t(e0), t(pol), t(az))


# (hits, nodes) given: too few of both, of hits only, of nodes only
@pytest.mark.parametrize("room", [(8, 8), (8, 1 << 22), (1 << 22, 8)])
@pytest.mark.parametrize("outputs,sched", [(H | K | T, None), (H | K | T, (3, 1)), (H | I | K | T, None),
                                           (H | I | K | T, (2, 0))])
def test_grown_arrays_match_oracle(outputs, sched, room):
    print(f"placed again: outputs {outputs}, schedule {sched}, room {room}", flush=True)
    w = workloads.WORKLOADS["e1to100_20planes_img32_100k"]
    geom = workloads.geometry(w)
    for n in (5, 300):
        host, dev = ics(w, n)
        sim = supa.Simulator(geom, outputs)
        if sched:
            sim.set_schedule(*sched)
        out = sim.simulate(*dev, w.seed, hit_capacity=room[0], node_capacity=room[1])
        ms = sim.timing()
        assert ms[2] >= ms[0] > 0 and ms[3] > 0 and ms[4] > 0, ms
        ref = O.simulate(geom, *host, w.seed)
        parity.check_all(parity.to_numpy(out), ref, geom, images=bool(outputs & I), tree=True)


def test_nothing_to_place_again():
    w = workloads.WORKLOADS["e10_normal_5planes_1k"]
    geom = workloads.geometry(w)
    _, dev = ics(w, 100)
    sim = supa.Simulator(geom, H)
    lib = sim.lib

    def again(out):
        _, o = sim._marshal(*dev, out, None, None, 0)
        st = lib.supa_place_again(sim.ctx, C.byref(o))
        sim._totals(out, o)
        return st

    big = sim.allocate(100, 1 << 16)
    assert again(big) == 5                                   # STATE: no call yet
    small = sim.allocate(100, 4)
    assert sim.run(*dev, 1, small) == 3
    total = small["total_hits"]
    assert total > 4
    assert again(sim.allocate(100, 4)) == 3                  # still too small
    out = dict(sim.allocate(0, total), **{k: small[k] for k in ("ledger", "counts", "hit_offsets")})
    assert again(out) == 0 and out["total_hits"] == total
    assert again(out) == 5                                   # done
    assert sim.run(*dev, 1, small) == 3
    assert sim.run(*dev, 2, big) == 0
    assert again(big) == 5                                   # another call since
    ref = sim.simulate(*dev, 1, hit_capacity=1 << 16)
    for k in ("hit_x", "hit_y", "hit_e"):
        assert torch.equal(out[k][:total].sort()[0], ref[k].sort()[0])
    assert torch.equal(out["hit_offsets"], ref["hit_offsets"])
