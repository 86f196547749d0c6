"""Shape variables by one wave per shower (small batches, and larger ones of
64 and more hits per shower) and by one lane per shower (larger batches of
fewer): segments at the edges of the read steps (256 hits) and tiles (768),
runs that cross them, one-hit runs, hits of layer -1, unaligned segments, an
array that ends with the last segment, and showers in error.

Against the shape oracle, at the bars of test_gpu_shapes (double-precision
sums; float results)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2202_05012_amd import shapes as SH
from tests.test_gpu_shapes import _t, check_shapes, oracle_shapes

pytestmark = pytest.mark.gpu

SIZES = [0, 1, 2, 3, 4, 5, 63, 64, 65, 255, 256, 257, 511, 513, 767, 768, 769, 1023, 1025,
         1535, 1536, 1537, 2303, 2305, 4000, 0, 1]


def layers(rng, m, L, kind):
    if kind == 0:                                      # one run
        lay = np.full(m, rng.integers(0, L))
    elif kind == 1:                                    # one-hit runs, then a long one
        lay = np.minimum(np.arange(m), L - 1)
    else:
        nl = int(rng.integers(1, L + 1))
        cuts = np.sort(rng.integers(0, m + 1, nl - 1))
        lay = np.repeat(rng.permutation(L)[:nl], np.diff(np.concatenate([[0], cuts, [m]])))
    lay = lay.astype(np.int32)
    if kind == 3:                                      # hits outside of the layers
        lay[rng.random(m) < 0.1] = -1
    if kind == 4:
        lay[-1:] = -1
        lay[:m // 2] = -1
    return lay


# (showers added, hits of each): by wave, by lane, by wave with several showers per wave
@pytest.mark.parametrize("more,hits", [(0, 0), (17000, 0), (40000, 70)])
@pytest.mark.parametrize("L", [1, 20, 64])
def test_segments_at_the_edges(more, hits, L):
    print(f"shapes: {more} more showers of {hits} hits, {L} layers", flush=True)
    rng = np.random.default_rng(100 * L + more + hits)
    lays = [layers(rng, m, L, k) for k in range(5) for m in SIZES]
    good = len(lays)
    lays.append(np.array([0] * 800 + [L] * 3, np.int32))             # out of range
    if L > 2:
        lays.append(np.array([1] * 700 + [2] * 300 + [1] * 5, np.int32))   # twice, in two tiles
        lays.append(np.tile([0, 1], 500).astype(np.int32))           # more runs than layers
    bad = len(lays) - good
    lays += [np.full(hits, L // 2, np.int32)] * more
    n = len(lays)
    cnt = np.array([len(v) for v in lays], np.int32)
    gap = rng.integers(0, 4, n)
    gap[good + bad:] = 0
    off = (np.cumsum(gap + cnt) - cnt).astype(np.int64)
    total = int(off[-1] + cnt[-1])
    x, y, e, lay = (np.full(total, v, t) for v, t in ((7e7, np.float32), (-7e7, np.float32),
                                                      (1e9, np.float32), (999, np.int32)))
    sid = np.full(total, -1, np.int64)
    px, py = rng.normal(3, 2, (2, max(hits, 1))).astype(np.float32)
    pe = rng.exponential(1, max(hits, 1)).astype(np.float32)
    for s in range(n):
        a, m = off[s], cnt[s]
        lay[a:a + m], sid[a:a + m] = lays[s], s
        if s < good + bad:
            x[a:a + m] = rng.normal(10, 3, m)
            y[a:a + m] = rng.normal(-5, 3, m)
            e[a:a + m] = rng.exponential(1, m)
        else:
            x[a:a + m], y[a:a + m], e[a:a + m] = px[:m], py[:m], pe[:m]
    args = [_t(v) for v in (off, cnt, x, y, e, lay)]
    lv, sv = SH.shower_shapes(*args, L, check=False)
    with pytest.raises(ValueError, match=f"{bad} showers"):
        SH.shower_shapes(*args, L)
    sel = np.r_[0:good, good + bad:min(n, good + bad + 1)]           # the added ones are all alike
    pos = np.full(n, -1)
    pos[sel] = np.arange(len(sel))
    new = np.where(sid >= 0, pos[sid], -1)
    new[sid < 0] = -1
    rlv, rsv = oracle_shapes(len(sel), L, new, lay, x, y, e)
    it = torch.from_numpy(sel).cuda()
    check_shapes(lv[it], sv[it], rlv, rsv)
    assert torch.isnan(lv[good:good + bad]).all() and torch.isnan(sv[good:good + bad]).all()
    a, b = lv[good + bad:], sv[good + bad:]
    if more:
        assert torch.equal(a.view(torch.int32), a[:1].view(torch.int32).expand_as(a))
        assert torch.equal(b.view(torch.int32), b[:1].view(torch.int32).expand_as(b))


def test_energies_that_are_not_numbers():
    """Both kernels give the same records where energies are NaN or infinite:
    the energy ratio exactly (no sums), the rest NaN in the same places."""
    print("shapes: NaN and infinite energies", flush=True)
    rng = np.random.default_rng(5)
    L, n, m = 8, 60, 900
    lay = np.sort(rng.integers(0, L, (n, m)), 1).astype(np.int32)
    x, y = rng.normal(1, 2, (2, n, m)).astype(np.float32)
    e = rng.exponential(1, (n, m)).astype(np.float32)
    e[rng.random((n, m)) < 0.004] = np.nan
    e[::7][rng.random((len(range(0, n, 7)), m)) < 0.002] = np.inf
    e[3] = np.nan
    res = []
    for more in (0, 17000):                                          # by wave, by lane
        off = np.concatenate([np.arange(n) * m, np.full(more, n * m)]).astype(np.int64)
        cnt = np.concatenate([np.full(n, m), np.zeros(more)]).astype(np.int32)
        lv, sv = SH.shower_shapes(*[_t(v) for v in (off, cnt, x.ravel(), y.ravel(), e.ravel(), lay.ravel())], L)
        res.append((lv[:n].cpu().numpy(), sv[:n].cpu().numpy()))
    ratio = SH.LAYER_VARS.index("energy_ratio")
    np.testing.assert_array_equal(res[0][0][..., ratio], res[1][0][..., ratio])
    assert np.isnan(res[0][0][..., ratio]).any() and np.isfinite(res[0][0][..., ratio]).any()
    for a, b in zip(*res):
        np.testing.assert_array_equal(np.isnan(a), np.isnan(b))
        np.testing.assert_array_equal(np.isinf(a), np.isinf(b))
