"""The judge's column sort and exact W1 at the edges of its tiles (8,192 keys)
and of its two ways to find a tile's starts (up to 128 tiles summed by the
scatter itself), against numpy.  Sorting moves bit patterns: exact.  W1 sums
doubles in another order than numpy: 1e-12 relative."""
import numpy as np
import pytest
import torch

from paper_2202_05012_amd import surrogate as S

pytestmark = pytest.mark.gpu


def sample(n, cols, seed):
    rng = np.random.default_rng(seed)
    x = rng.normal(0.0, 1.0, (n, cols)).astype(np.float32)
    kinds = [lambda c: c, lambda c: np.rint(20 * np.abs(c)), lambda c: np.full_like(c, 2.5),
             lambda c: c * np.float32(1e30), lambda c: np.where(c > 1, np.inf, np.where(c < -1, -np.inf, c * 0))]
    for c in range(cols):
        x[:, c] = kinds[c % len(kinds)](x[:, c])
    return x


def key(x):
    u = np.ascontiguousarray(x).view(np.uint32)
    return np.where(u >> 31, ~u, u | 0x80000000)


@pytest.mark.parametrize("n,cols", [(1, 1), (63, 3), (64, 33), (65, 5), (8191, 2), (8192, 3), (8193, 5), (20011, 40),
                                    (128 * 8192, 2), (128 * 8192 + 1, 2), (1_100_007, 3)])
def test_sort_and_w1_at_tile_edges(n, cols):
    print(f"sort: {n} x {cols}", flush=True)
    a, b = sample(n, cols, 1), sample(n, cols, 2)
    if n > 100:
        a[7, 0] = np.nan
    got = S.sort_columns(torch.from_numpy(a).cuda()).cpu().numpy()
    want = np.sort(key(a), axis=0).T
    assert np.array_equal(key(got), want)
    fin = [c for c in range(cols) if c % 5 != 4]
    if n > 100:
        a[7, 0] = 0.0
    w1 = S.w1_equal(torch.from_numpy(a[:, fin].copy()).cuda(), torch.from_numpy(b[:, fin].copy()).cuda()).cpu().numpy()
    ref = np.abs(np.sort(a[:, fin], 0).astype(np.float64) - np.sort(b[:, fin], 0)).mean(0)
    np.testing.assert_allclose(w1, ref, rtol=1e-12, atol=0)


def test_rows_with_a_leading_dimension():
    x = torch.from_numpy(sample(3001, 12, 3)).cuda()
    L = S._lib()
    wb = int(L.supa_sort_columns_workspace_bytes(3001, 5))
    work, out = torch.empty(wb + 4, dtype=torch.uint8, device="cuda"), torch.empty((5, 3001), device="cuda")
    S._check(L.supa_sort_columns(S._stream(), 3001, 5, x.data_ptr() + 8, 12, out.data_ptr(), work.data_ptr() + 4, wb))
    assert np.array_equal(key(out.cpu().numpy()), np.sort(key(x.cpu().numpy()[:, 2:7]), 0).T)
