"""Weight and bias gradients of the surrogate's convolution at the edges of the
work items of their kernels, against the FP64 reference.

Tolerance 2e-5 of the largest value: FP32 sums of at most 1e4 products of
values of unit size, as in the other gradient checks.
"""
import numpy as np
import pytest

from oracle import conv_ref as cr
from tests.conftest import announce

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
sur = pytest.importorskip("paper_2306_11320_amd.surrogate")


def t_bf16(a):
    return torch.tensor(np.asarray(a, np.float32), device="cuda").to(torch.bfloat16).contiguous()


def weight_grad(dy, x, cin, relu_in, groups, dil):
    stream = torch.cuda.current_stream()
    part = torch.full((groups * 32 * 9 * cin,), float("nan"), device="cuda")
    out = torch.full((32, 9, cin), float("nan"), device="cuda")
    sur.sur_weight_grad(dy, x, cin, relu_in, part, groups, out, stream, dil)
    torch.cuda.synchronize()
    return out.cpu().numpy().astype(np.float64)


# items of 8 rows (of one residue class mod dil) x 64 pixels; windows of 96
# pixels up to dilation 16 and of 192 beyond, in three pieces above 64
@pytest.mark.parametrize("cin", [8, 32])
@pytest.mark.parametrize("dil,H,W,groups", [(1, 1, 1, 1), (1, 8, 64, 3), (1, 9, 65, 256), (2, 17, 63, 2), (3, 25, 79, 7),
                                            (16, 19, 17, 5), (16, 40, 130, 64), (17, 18, 66, 4), (64, 66, 64, 9),
                                            (65, 9, 70, 2), (100, 201, 129, 31)])
def test_weight_gradient_edges(cin, dil, H, W, groups):
    announce("weight_gradient_edges", cin, dil, H, W, groups)
    rng = np.random.default_rng(1000 * cin + 10 * dil + W)
    N = 2 if H < 100 else 1
    a = cr.bf16_round(rng.standard_normal((N, H, W, cin)))
    g = cr.bf16_round(rng.standard_normal((N, H, W, 32)))
    for relu_in in (False, True):
        ref = cr.conv_weight_grad(g, cr.relu(a) if relu_in else a, dil)
        got = weight_grad(t_bf16(g), t_bf16(a), cin, relu_in, groups, dil)
        assert np.abs(got - ref).max() <= 2e-5 * np.abs(ref).max()


def test_weight_gradient_unaligned_and_not_a_number():
    """Operands at an odd element of their storage; the ReLU takes NaN inputs as zero."""
    announce("weight_gradient_unaligned")
    rng = np.random.default_rng(8)
    N, H, W, dil = 1, 11, 70, 4
    a = cr.bf16_round(rng.standard_normal((N, H, W, 32)))
    g = cr.bf16_round(rng.standard_normal((N, H, W, 32)))

    def odd(v):
        s = torch.zeros(v.size + 1, dtype=torch.bfloat16, device="cuda")
        s[1:] = t_bf16(v).reshape(-1)
        return s[1:].view(v.shape)
    bad = a.copy()
    bad[0, 3, 5, ::3] = np.nan
    bad[0, 10, 69, 1::2] = -np.nan
    ref = cr.conv_weight_grad(g, np.where(bad > 0, bad, 0.0), dil)
    got = weight_grad(odd(g), odd(bad), 32, True, 6, dil)
    assert np.abs(got - ref).max() <= 2e-5 * np.abs(ref).max()


@pytest.mark.parametrize("cin,W,dil,relu_in", [(32, 70, 4, True), (8, 65, 1, False), (32, 41, 16, False), (32, 127, 20, True)])
def test_weight_gradient_infinite_input(cin, W, dil, relu_in):
    """An infinite input gives infinities of the reference's signs, never NaN:
    dy counts nothing beyond its row, whose columns meet real (periodic) inputs."""
    announce("weight_gradient_infinite", cin, W, dil, relu_in)
    rng = np.random.default_rng(W)
    a = cr.bf16_round(rng.standard_normal((1, 45, W, cin)))
    g = cr.bf16_round(rng.standard_normal((1, 45, W, 32)))
    a[0, 22, 3, 1] = np.inf
    if not relu_in:
        a[0, 22, W - 1, 6] = -np.inf
    with np.errstate(invalid="ignore"):
        ref = cr.conv_weight_grad(g, cr.relu(a) if relu_in else a, dil)
    got = weight_grad(t_bf16(g), t_bf16(a), cin, relu_in, 5, dil)
    inf = np.isinf(ref)
    assert inf.sum() >= 9 * 32 and not np.isnan(ref).any()
    assert np.array_equal(got[inf], ref[inf])
    assert np.abs(got[~inf] - ref[~inf]).max() <= 2e-5 * np.abs(ref[~inf]).max()


@pytest.mark.parametrize("npix,groups", [(1, 1), (1, 4), (63, 1), (64, 3), (1000, 5), (4097, 256)])
def test_bias_gradient_edges(npix, groups):
    announce("bias_gradient_edges", npix, groups)
    g = cr.bf16_round(np.random.default_rng(npix).standard_normal((1, 1, npix, 32)))
    part = torch.full((32 * groups,), float("nan"), device="cuda")
    out = torch.full((32,), float("nan"), device="cuda")
    sur.sur_bias_grad(t_bf16(g), part, groups, out, torch.cuda.current_stream())
    torch.cuda.synchronize()
    ref = g.sum(axis=(0, 1, 2))
    assert np.abs(out.cpu().numpy() - ref).max() <= 2e-5 * max(1.0, np.abs(ref).max())


@pytest.mark.parametrize("H,W,dil", [(1, 1, 1), (9, 33, 1), (17, 31, 3), (40, 64, 16), (8, 130, 16), (73, 16, 5)])
def test_packed_first_layer_equals_pack_then_conv(H, W, dil):
    """The first layer that packs the state as it reads it, bit by bit."""
    announce("packed_first_layer", H, W, dil)
    rng = np.random.default_rng(H + W)
    stream = torch.cuda.current_stream()
    f = {k: torch.tensor(rng.standard_normal((H, W)), dtype=torch.float32, device="cuda") for k in sur.FIELDS}
    sc = sur.SurScales(0.3, 1.7, 0.1, 0.02, 0.6, 0.35, -0.2, (sur.C.c_float * 5)(*[1.0] * 5))
    w, b = t_bf16(0.2 * rng.standard_normal((32, 9, 8))), torch.tensor(rng.standard_normal(32), device="cuda").float()
    x = torch.empty((1, H, W, 8), dtype=torch.bfloat16, device="cuda")
    ref = torch.empty((1, H, W, 32), dtype=torch.bfloat16, device="cuda")
    got = torch.full_like(ref, float("nan"))
    sur.sur_pack(f, sc, x, stream)
    sur.sur_conv3x3(x, 8, w, b, None, None, ref, False, stream, dil)
    sur.sur_pack_conv3x3(f, sc, w, b, got, stream, dil)
    torch.cuda.synchronize()
    assert torch.equal(ref.view(torch.int16), got.view(torch.int16))


@pytest.mark.parametrize("N,H,W,dil,relu_in", [(1, 1, 1, 1, True), (2, 9, 33, 1, True), (1, 30, 95, 7, False),
                                               (3, 64, 64, 16, True), (4, 70, 129, 1, True)])
def test_output_layer_with_squared_error(N, H, W, dil, relu_in):
    """The output layer that compares its increment with the target: gradient
    bitwise that of the two kernels, loss within FP32 summation error."""
    announce("conv_mse", N, H, W, dil)
    rng = np.random.default_rng(N + H + W)
    stream = torch.cuda.current_stream()
    x, w = t_bf16(rng.standard_normal((N, H, W, 32))), t_bf16(0.2 * rng.standard_normal((32, 9, 32)))
    b = torch.tensor(rng.standard_normal(32), device="cuda").float()
    target = torch.tensor(rng.standard_normal((N, H, W, 5)), device="cuda").float()
    delta = torch.empty((N, H, W, 32), device="cuda")
    ref = torch.empty((N, H, W, 32), dtype=torch.bfloat16, device="cuda")
    got = torch.full_like(ref, float("nan"))
    part, lpart = torch.empty(64, device="cuda"), torch.full((sur.LOSS_PARTS,), float("nan"), device="cuda")
    sur.sur_conv3x3(x, 32, w, b, None, None, delta, relu_in, stream, dil)
    sur.sur_mse(delta, target, 0.37, ref, part, stream)
    sur.sur_conv3x3_mse(x, w, b, relu_in, target, 0.37, got, lpart, stream, dil)
    torch.cuda.synchronize()
    assert torch.equal(ref.view(torch.int16), got.view(torch.int16))
    exact = float(((delta[..., :5].double() - target.double()) ** 2).sum())
    assert abs(float(lpart.double().sum()) - exact) <= 1e-5 * exact


@pytest.mark.parametrize("cin,H,W,dil,groups", [(8, 5, 30, 1, 1), (32, 9, 65, 2, 3), (32, 40, 70, 16, 20),
                                                (32, 18, 66, 17, 9), (8, 24, 64, 1, 64)])
def test_layer_gradients_and_adam(cin, H, W, dil, groups):
    """Partial sums of a layer's gradients into Adam: weights bitwise as by the
    separate kernels (the same sums in the same order where every group has an
    item), biases within FP32 summation error."""
    announce("layer_grads_adam", cin, H, W, dil, groups)
    rng = np.random.default_rng(cin + H + W)
    stream = torch.cuda.current_stream()
    N = 2
    g = cr.bf16_round(rng.standard_normal((N, H, W, 32)))
    dy, x = t_bf16(g), t_bf16(rng.standard_normal((N, H, W, cin)))

    def f32(*shape):
        return torch.tensor(rng.standard_normal(shape), device="cuda").float()
    W0, b0, m1, m2, mb1, mb2 = f32(32, 9, cin), f32(32), f32(32, 9, cin), f32(32, 9, cin) ** 2, f32(32), f32(32) ** 2
    Wr, m1r, m2r = W0.clone(), m1.clone(), m2.clone()
    Wb, Wbr = torch.empty_like(W0, dtype=torch.bfloat16), torch.empty_like(W0, dtype=torch.bfloat16)
    part = torch.full((groups * (32 * 9 * cin + 32),), float("nan"), device="cuda")
    gw = torch.empty_like(W0)
    lpart, loss = f32(sur.LOSS_PARTS), torch.empty(1, device="cuda")
    b1 = mb1.clone()
    sur.sur_layer_grads(dy, x, cin, cin == 32, part, groups, stream, dil)
    sur.sur_adam_layers([(part, W0, b0, m1, m2, mb1, mb2, Wb, cin, groups)], 1e-2, 3, lpart, loss, stream)
    wpart = torch.empty(groups * 32 * 9 * cin, device="cuda")
    sur.sur_weight_grad(dy, x, cin, cin == 32, wpart, groups, gw, stream, dil)
    sur.sur_adam(Wr, gw, m1r, m2r, Wbr, 1e-2, 3, stream)
    torch.cuda.synchronize()
    for a, b in ((W0, Wr), (m1, m1r), (m2, m2r), (Wb.float(), Wbr.float())):
        assert torch.equal(a, b)
    ref = g.sum(axis=(0, 1, 2))
    got = (mb1.double() - 0.9 * b1.double()).cpu().numpy() / 0.1
    assert np.abs(got - ref).max() <= 2e-5 * np.abs(ref).max() + 1e-5
    assert abs(float(loss) - float(lpart.double().sum())) <= 1e-5 * float(lpart.abs().sum())
