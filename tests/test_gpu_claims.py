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
