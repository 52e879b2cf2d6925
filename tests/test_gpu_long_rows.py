"""Convolutions on rows whose byte offsets pass 32 bits: 64 bytes a pixel for
32 channels, 16 for 8, from 2^26 and 2^28 pixels on.

The frame is zero but for its first and last pixels, whose neighbourhoods (and
the same places of a row shorter by the offsets' period) are compared with
the FP64 reference on the few pixels around the seam.  Tolerance: one BF16
step of the reference rounded to BF16, as in the other convolution checks.
"""
import numpy as np
import pytest

from oracle import conv_ref as cr
from tests.conftest import announce

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
sur = pytest.importorskip("paper_2306_11320_amd.surrogate")

E = 160          # pixels kept at either end


def t_bf16(a):
    return torch.tensor(np.asarray(a, np.float32), device="cuda").to(torch.bfloat16).contiguous()


def ends(t, lo, hi):
    """Pixels [lo, lo + E) and [hi, hi + E) of the row."""
    return [t[0, 0, q:q + E].float().cpu().numpy().astype(np.float64) for q in (lo, hi)]


def frame(rng, cin):
    """A row of the seam's pixels alone: the last E, then the first E."""
    return cr.bf16_round(rng.standard_normal((1, 1, 2 * E, cin)))


@pytest.mark.parametrize("cin,dil", [(8, 1), (8, 16), (32, 4), (32, 16), (32, 17)])
def test_conv_row_past_32_bit_offsets(cin, dil):
    W = (1 << 32) // (2 * cin) + 100
    announce("conv_long_row", cin, dil, W)
    rng = np.random.default_rng(cin + dil)
    seam = frame(rng, cin)
    w, b = cr.bf16_round(0.2 * rng.standard_normal((32, 9, cin))), rng.standard_normal(32).astype(np.float32)
    x = torch.zeros((1, 1, W, cin), dtype=torch.bfloat16, device="cuda")
    x[0, 0, W - E:] = t_bf16(seam[0, 0, :E])
    x[0, 0, :E] = t_bf16(seam[0, 0, E:])
    out = torch.empty((1, 1, W, 32), dtype=torch.bfloat16, device="cuda")
    sur.sur_conv3x3(x, cin, t_bf16(w), torch.tensor(b, device="cuda"), None, None, out, False,
                    torch.cuda.current_stream(), dil)
    torch.cuda.synchronize()
    # the reference on the seam with zeros around it; E - 2 dil pixels of each end see only those
    pad = np.zeros((1, 1, 64, cin))
    ref = cr.bf16_round(cr.conv(np.concatenate([pad, seam, pad], axis=2), w, b, dil))[0, 0, 64:64 + 2 * E]
    first, last = ends(out, 0, W - E)
    for got, r in ((last, ref[:E]), (first, ref[E:])):
        assert np.all(np.abs(got - r) <= 2 ** -7 * np.abs(r) + 1e-6)
    del x, out
    torch.cuda.empty_cache()


@pytest.mark.parametrize("vol", [False, True])
def test_output_layer_row_past_32_bit_offsets(vol):
    W, dil = (1 << 26) + 100, 8
    announce("advance_long_row", vol, W)
    rng = np.random.default_rng(3)
    seam = frame(rng, 32)
    w, b = cr.bf16_round(0.2 * rng.standard_normal((32, 9, 32))), rng.standard_normal(32).astype(np.float32)
    x = torch.zeros((1, 1, W, 32), dtype=torch.bfloat16, device="cuda")
    x[0, 0, W - E:] = t_bf16(seam[0, 0, :E])
    x[0, 0, :E] = t_bf16(seam[0, 0, E:])
    f = {k: torch.zeros((1, W), device="cuda") for k in sur.FIELDS}
    sc = sur.SurScales(0.3, 1.7, 0.1, 0.02, 0.6, 0.35, -0.2, (sur.C.c_float * 5)(*[0.5] * 5))
    stream = torch.cuda.current_stream()
    bd = torch.tensor(b, device="cuda")
    if vol:
        part, v = torch.zeros(8 * sur.VOLUME_PARTS, dtype=torch.float64, device="cuda"), torch.zeros(1, dtype=torch.float64, device="cuda")
        sur.sur_conv3x3_advance_volume(x, t_bf16(w), bd, True, sc, f, part, v, stream, dil)
    else:
        sur.sur_conv3x3_advance(x, t_bf16(w), bd, True, sc, f, stream, dil)
    torch.cuda.synchronize()
    pad = np.zeros((1, 1, 64, 32))
    ref = 0.5 * cr.conv(np.concatenate([pad, cr.relu(seam), pad], axis=2), w, b, dil)[0, 0, 64:64 + 2 * E, :5]
    for c, k in enumerate(sur.FIELDS):
        got = f[k][0].cpu()
        got = np.concatenate([got[W - E:], got[:E]]).astype(np.float64)
        assert np.abs(got - ref[:, c]).max() <= 2e-5 * np.abs(ref).max(), k
    if vol:
        exact = float((0.5 * (1.0 - f["phi"].double())).sum())
        assert abs(float(v) - exact) <= 1e-12 * abs(exact)
    del x, f
    torch.cuda.empty_cache()
