"""Sums of the fused final layer's tiles, sixteen to sixty-four lanes per
shower by the number of layers, and the head's gate (rows staged without
divisions), at the layer counts where the lanes per shower change and with
rows that leave the last workgroup ragged.

The fused layer against the unfused product and gate: the products differ by
float accumulation (bar of test_gpu_surrogate: 2e-4).  The head's gate against
the oracle with zero spread (rho < 0: energies are the means scaled by
e0 / y_scale, two roundings) and its score (three: 1e-5)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import surrogate_oracle as SO
from paper_2202_05012_amd import surrogate as S
from tests.test_gpu_surrogate import bf16_round, dev16

pytestmark = pytest.mark.gpu

LAYERS = [1, 2, 15, 16, 17, 31, 32, 33, 63, 64]


@pytest.mark.parametrize("rho", [-1.0, 0.4])
@pytest.mark.parametrize("L", LAYERS)
def test_tile_sums(L, rho):
    print(f"gate: {L} layers of 128 bins, rho {rho}", flush=True)
    rng = np.random.default_rng(L)
    B, K, D = 131, 64, 128 * L
    h = bf16_round(rng.normal(size=(B, K)))
    W = (rng.normal(size=(K, 2 * D)) * 0.1).astype(np.float32)
    bias = (rng.normal(size=2 * D) * 0.1).astype(np.float32)
    bias[:D] += 1.0
    e0 = torch.from_numpy(rng.uniform(1, 100, B).astype(np.float32)).cuda()
    tb, th = torch.from_numpy(bias).cuda(), dev16(h)
    wt = S.transpose_to_bf16(torch.from_numpy(W).cuda())
    le, unc, cnt = S.gate_fused(th, wt, tb, e0, L, rho=rho, seed=9, row_base=2 ** 32 - 50, cnt_thr=1e-3)
    # (the plain product takes multiples of eight rows)
    rows = torch.zeros((136, K), dtype=th.dtype, device="cuda")
    rows[:B] = th
    out = torch.empty((136, 2 * D), dtype=torch.float32, device="cuda")
    S.gemm(rows, dev16(bf16_round(W)), out, 0, 0, 1, bias=tb)
    ref_le, ref_unc, _ = S.gate(out[:B], e0, L, rho=rho, seed=9, row_base=2 ** 32 - 50)
    np.testing.assert_allclose(le.cpu().numpy(), ref_le.cpu().numpy(), rtol=2e-4, atol=1e-5)
    np.testing.assert_allclose(unc.cpu().numpy(), ref_unc.cpu().numpy(), rtol=2e-4)
    assert ((cnt >= 0) & (cnt <= 128)).all() and (cnt == cnt.round()).all()


@pytest.mark.parametrize("B", [1, 63, 64, 65, 200])
@pytest.mark.parametrize("L", LAYERS)
def test_head_gate_rows(L, B):
    print(f"head gate: {B} rows of {L} layers", flush=True)
    rng = np.random.default_rng(1000 * L + B)
    out = np.concatenate([rng.uniform(0.1, 3, (B, L)), rng.uniform(-9, 3, (B, L))], 1).astype(np.float32)
    e0 = rng.uniform(1, 100, B).astype(np.float32)
    le, unc, _ = S.gate(torch.from_numpy(out).cuda(), torch.from_numpy(e0).cuda(), L, y_scale=20.0)
    ref_le, ref_unc = SO.gate(out, e0, L, 20.0, S.S_CLAMP, -1.0, 0, 0)
    np.testing.assert_allclose(le.cpu().numpy(), ref_le, rtol=4e-7)
    np.testing.assert_allclose(unc.cpu().numpy(), ref_unc, rtol=1e-5)
