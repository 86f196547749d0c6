"""First showers by position, later ones from the work counter: batch sizes
around the grid (4,096 waves by default; 1 to 4 showers per wave at first),
against the oracle."""
import numpy as np
import pytest
import torch

from oracle import supa_oracle as O
from paper_2202_05012_amd import supa, workloads
from tests import parity

pytestmark = pytest.mark.gpu


def dev_t(a):
    return torch.from_numpy(np.ascontiguousarray(a, np.float32)).cuda()


@pytest.mark.parametrize("n", [1, 2, 4095, 4097, 8193, 12289, 16384, 16385, 20011])
def test_batches_around_the_grid(n):
    w = workloads.WORKLOADS["e10_normal_5planes_1k"]
    geom = workloads.geometry(w)
    rng = np.random.default_rng(n)
    e0 = rng.uniform(0.05, 1.5, n).astype(np.float32)       # some below the threshold at once
    pol = rng.uniform(0.0, 0.2, n).astype(np.float32)
    az = rng.uniform(0.0, 6.28, n).astype(np.float32)
    print(f"claims: {n} showers", flush=True)
    sim = supa.Simulator(geom, supa.OUT_HITS | supa.OUT_TREE | supa.OUT_KEYS)
    ref = O.simulate(geom, e0, pol, az, 7)
    for _ in range(2):                                      # the counters start afresh on each call
        out = parity.to_numpy(sim.simulate(dev_t(e0), dev_t(pol), dev_t(az), 7))
        parity.check_all(out, ref, geom, tree=True)
    assert int(out["total_steps"]) == int(ref["counts"][:, 2].sum())


@pytest.mark.parametrize("waves_per_cu,sub_batches", [(1, 1), (1, 3), (16, 2)])
def test_few_waves_and_sub_batches(waves_per_cu, sub_batches):
    w = workloads.WORKLOADS["e10_normal_5planes_1k"]
    geom = workloads.geometry(w)
    n = 3001
    e0, pol, az = (np.ascontiguousarray(a) for a in workloads.initial_conditions(w, n))
    print(f"claims: {waves_per_cu} waves per CU, {sub_batches} sub-batches", flush=True)
    sim = supa.Simulator(geom, supa.OUT_HITS | supa.OUT_KEYS, waves_per_cu=waves_per_cu, sub_batches=sub_batches)
    out = parity.to_numpy(sim.simulate(dev_t(e0), dev_t(pol), dev_t(az), w.seed))
    parity.check_all(out, O.simulate(geom, e0, pol, az, w.seed), geom)


@pytest.mark.parametrize("n,e,planes", [(1, 1000.0, 20), (3, 900.0, 9), (63, 300.0, 12), (130, 250.0, 20), (600, 60.0, 20),
                                        (1024, 40.0, 8)])
def test_dealt_out_showers(n, e, planes):
    """Automatic subtree items: showers dealt out at 256 pending particles
    (and those that never reach them), few planes, 1 to 1,024 showers."""
    w = workloads.WORKLOADS["loge1to1000_20planes_1m"]
    geom = workloads.geometry(w, n_planes=planes)
    _, pol, az = workloads.initial_conditions(w, n)
    e0 = np.full(n, e, np.float32)
    e0[::7] *= 0.05
    print(f"claims: items, {n} showers of {e}, {planes} planes", flush=True)
    ref = O.simulate(geom, e0, pol, az, 11)
    for outputs in (supa.OUT_HITS | supa.OUT_TREE | supa.OUT_KEYS, supa.OUT_HITS | supa.OUT_KEYS, 0):
        sim = supa.Simulator(geom, outputs)
        out = parity.to_numpy(sim.simulate(dev_t(e0), dev_t(pol), dev_t(az), 11))
        parity.check_counts(out, ref)
        if outputs:
            parity.check_all(out, ref, geom, tree=bool(outputs & supa.OUT_TREE))
        items = sim.subtree_counts()["items"][0]
        if planes <= 8:
            assert items == 0
        if planes == 20 and e0.max() >= 250.0:
            assert items > 0
