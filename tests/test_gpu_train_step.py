"""The fused training step against the layer-by-layer products (forward,
loss gradient, backward, Adam), which tests/test_gpu_surrogate.py checks
against the float64 oracle: both round the same quantities to bf16, so they
differ by the order of float32 sums and by the bf16 values that this moves
across a rounding boundary.  A sum of up to 10^4 terms is off by about 1e-6,
so about 1e-6 / 2^-9 = 5e-4 of the bf16 values flip by 2^-8: sqrt(5e-4) 2^-8 =
9e-5 per tensor and layer.  Bound: 1e-3 in the 2-norm."""
import numpy as np
import pytest
import torch

from paper_2202_05012_amd import surrogate as S

pytestmark = pytest.mark.gpu


def data(B, k_in, D, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    x = torch.zeros(B, k_in, device="cuda")
    x[:, :min(k_in, 19)] = torch.randn(B, min(k_in, 19), generator=g, device="cuda")
    e0 = 1.0 + 99.0 * torch.rand(B, generator=g, device="cuda")
    img = torch.rand(B, D, generator=g, device="cuda") * (torch.rand(B, D, generator=g, device="cuda") < 0.3)
    return S.to_bf16(x), img * e0[:, None] / 20.0, e0


def layer_by_layer(net, x, img, e0, lr, s_clamp, mse_mean, y_scale):
    out, acts, pres = net.forward(x, keep=True)
    B, D = out.shape[0], out.shape[1] // 2
    dout = torch.empty(out.shape, dtype=torch.int16, device="cuda")
    loss = torch.zeros(1, device="cuda")
    S._check(S._lib().supa_nll_grad(S._stream(), B, D, S._p(out), S._p(img), S._p(e0), y_scale, s_clamp,
                                    1 if mse_mean else 0, S._p(dout), S._p(loss)))
    dWs, dbs = net.backward(acts, pres, dout)
    net.adam(dWs, dbs, lr=lr)
    return loss / (B * D)


def rel(a, b):
    a, b = a.double(), b.double()
    return float((a - b).norm() / max(float(b.norm()), 1e-30))


@pytest.mark.parametrize("B,dims,s_clamp,mse_mean", [
    (8, [32, 256, 40], 20.0, False),                          # one hidden layer, one row block
    (40, [16, 256, 256, 8], 20.0, True),                      # the fewest inputs and outputs
    (256, [256, 256, 256, 256, 128], 20.0, True),             # the most inputs, whole tiles
    (264, [32, 256, 256, 256, 256, 264], 0.5, False),         # ragged bins and rows, clamped log-variances
    (1032, [32, 256, 256, 256, 256, 1288], 0.0, True),        # several row parts, log-variances held
    (4104, [32, 256, 256, 256, 256, 10240], 20.0, True),      # the image model, ragged rows
])
def test_fused_step_matches_layer_by_layer(B, dims, s_clamp, mse_mean):
    print(f"train step: batch {B}, layers {dims}", flush=True)
    D, ys = dims[-1] // 2, 20.0
    x, img, e0 = data(B, dims[0], D, B)
    a, b = S.MLP(dims, seed=3), S.MLP(dims, seed=3)
    assert a._train_bytes(x, img) > 0
    for net in (a, b):
        net.step = 100
        for v in (*net.vW, *net.vb):
            v.fill_(1e-6)
    la = a.train_step(x, img, e0, lr=1e-3, s_clamp=s_clamp, mse_mean=mse_mean, y_scale=ys)
    lb = layer_by_layer(b, x, img, e0, 1e-3, s_clamp, mse_mean, ys)
    assert a.step == b.step == 101
    assert rel(la, lb) < 1e-5
    for l in range(len(dims) - 1):
        for name in ("mW", "mb", "vW", "vb", "W", "b"):
            assert rel(getattr(a, name)[l], getattr(b, name)[l]) < 1e-3, (l, name)
        assert (S.bf16_to_float(a.Wb[l]) - a.W[l]).abs().max() <= a.W[l].abs().max() * 2.0 ** -8
    if s_clamp == 0.0:                                        # held log-variances have no gradient
        assert float(a.mb[-1][D:].abs().max()) == 0.0


def test_unaligned_and_odd_networks_take_the_general_path():
    x, img, e0 = data(64, 32, 20, 1)
    net = S.MLP([32, 256, 40], seed=1)
    shifted = torch.empty(64 * 20 + 1, device="cuda")[1:].view(64, 20).copy_(img)
    assert net._train_bytes(x, shifted) < 0
    assert S.MLP([32, 128, 40], seed=1)._train_bytes(x, img) < 0
    other = S.MLP([32, 256, 40], seed=1)
    la, lb = net.train_step(x, img, e0), other.train_step(x, shifted, e0)
    assert rel(la, lb) < 1e-5
    with pytest.raises(Exception):
        net.train_step(x[:60], img[:60], e0[:60])             # 60 rows: not a multiple of 8
    assert net.step == 1


@pytest.mark.parametrize("part", ["forward", "backward", "adam"])
@pytest.mark.parametrize("how", ["subclass", "class", "network", "other network"])
def test_replaced_parts_of_the_step_are_called(part, how, monkeypatch):
    """A part replaced on a subclass, on the class, on the network or by another
    network's method is what the step calls, as when it goes layer by layer."""
    x, img, e0 = data(64, 32, 20, 1)
    called = []
    plain = getattr(S.MLP, part)

    def replaced(self, *args, **kw):
        called.append(part)
        return plain(self, *args, **kw)
    cls = type("Sub", (S.MLP,), {part: replaced}) if how == "subclass" else S.MLP
    net, other = cls([32, 256, 40], seed=1), S.MLP([32, 256, 40], seed=1)
    if how == "class":
        monkeypatch.setattr(S.MLP, part, replaced)
    elif how == "network":
        setattr(net, part, lambda *args, **kw: replaced(net, *args, **kw))
    elif how == "other network":
        setattr(net, part, getattr(other, part))
        before = [w.clone() for w in (*net.W, *other.W)]
    net.train_step(x, img, e0)
    if how != "other network":
        assert called == [part]
    elif part == "adam":                                      # the other network is the one that is stepped
        assert (net.step, other.step) == (0, 1)
        assert [torch.equal(a, b) for a, b in zip(before, (*net.W, *other.W))] == [True, True, False, False]
    else:
        assert (net.step, other.step) == (1, 0)
    assert net._train_bytes(x, img) < 0


# (rows 3 and 60 of e0; bins of rows 5 and 61 of img), each a valid float of no use as an energy
@pytest.mark.parametrize("e", [None, np.inf, 0.0, 1e38, 3e38, 2.0 ** -126])
@pytest.mark.parametrize("t", [None, np.inf, -np.inf, np.nan, 3e38])
def test_targets_beyond_numbers_match_layer_by_layer(e, t):
    """Infinite, zero and huge energies, infinite and undefined targets: finite
    where the layer-by-layer step is, with the same infinities and NaN."""
    x, img, e0 = data(64, 32, 20, 1)
    img[3] = img[60] = 0.0 if e is None or e >= 1.0 else 1e-30
    if e is not None:
        e0[3] = e0[60] = float(e)
    if t is not None:
        img[5, 7] = img[61, 19] = float(t)
    a, b = S.MLP([32, 256, 256, 40], seed=1), S.MLP([32, 256, 256, 40], seed=1)
    assert a._train_bytes(x, img) > 0
    la = a.train_step(x, img, e0, s_clamp=5.0, mse_mean=True, y_scale=1.0)
    lb = layer_by_layer(b, x, img, e0, 1e-3, 5.0, True, 1.0)
    pairs = [(la, lb)] + [(getattr(a, k)[l], getattr(b, k)[l]) for k in ("mW", "mb", "W", "b") for l in range(3)]
    for p, q in pairs:
        assert torch.equal(p.isnan(), q.isnan())
        assert torch.equal(torch.where(p.isinf(), p, 0.0), torch.where(q.isinf(), q, 0.0))
        ok = q.isfinite()
        assert not bool(ok.any()) or rel(p[ok], q[ok]) < 1e-3


@pytest.mark.parametrize("B,dims", [
    (192, [32, 256, 256, 40]),                                # the first fold of partial sums, and around it
    (200, [32, 256, 256, 40]),
    (256, [256, 256, 256, 128]),
    (1032, [32, 256, 256, 256, 256, 1288]),
    (8192, [32, 256, 256, 256, 256, 40]),                     # the per-layer head
    (8192, [32, 256, 256, 256, 256, 10240]),                  # the image model
])
def test_gradients_no_further_from_float64_than_layer_by_layer(B, dims):
    """Weight and bias gradients (with b1 = 0 a step's first moments) against
    float64 products of the same bf16 values.  Weights: the root mean square
    error is no larger than that of the layer-by-layer products (the same sums
    up to 256 rows, then at most 320 rows in one accumulator where theirs has
    256 to 1,184).  Biases: at most 2 B / 192 + 12 roundings to 24 bits in a
    row (rows of a thread, 32 threads in pairs, parts)."""
    print(f"gradients: batch {B}, layers {dims}", flush=True)
    D, ys = dims[-1] // 2, 20.0
    x, img, e0 = data(B, dims[0], D, B)
    a, b = S.MLP(dims, seed=3), S.MLP(dims, seed=3)
    a._train_fused(x, img, e0, 1e-3, 20.0, False, ys, a._train_bytes(x, img), b1=0.0)
    out, acts, pres = b.forward(x, keep=True)
    dout = torch.empty(out.shape, dtype=torch.int16, device="cuda")
    loss = torch.zeros(1, device="cuda")
    S._check(S._lib().supa_nll_grad(S._stream(), B, D, S._p(out), S._p(img), S._p(e0), ys, 20.0, 0, S._p(dout),
                                    S._p(loss)))
    dWs, dbs = b.backward(acts, pres, dout)
    g = dout
    grads = [None] * len(dWs)
    for l in range(len(dWs) - 1, -1, -1):                     # (the values that b.backward went through)
        grads[l] = g
        if l > 0:
            gn = torch.empty((B, dims[l]), dtype=torch.int16, device="cuda")
            S.gemm(g, b.Wb[l], gn, trans_a=0, trans_b=1, epilogue=3, pre=pres[l - 1])
            g = gn
    rms = lambda m, ref: float((m.double() - ref).square().mean().sqrt())
    for l in range(len(dWs)):
        h, g = (S.bf16_to_float(t[l]).double() for t in (acts, grads))
        for name, one, two, ref in (("W", a.mW[l], dWs[l], h.t().contiguous() @ g), ("b", a.mb[l], dbs[l], g.sum(0))):
            err = [rms(t, ref) / rms(ref, 0.0) for t in (one, two)]
            print(f"  layer {l} {name}: {err[0]:.3g}, layer by layer {err[1]:.3g}", flush=True)
        assert rms(a.mW[l], h.t().contiguous() @ g) <= rms(dWs[l], h.t().contiguous() @ g), l
        assert bool(((a.mb[l].double() - g.sum(0)).abs() <= (B / 96 + 12) * 2.0 ** -24 * g.abs().sum(0)).all()), l
