"""Network layer kernels at the edges of their tiles (GPU).

Every layer gets the same bfloat16 operands as a 64-bit torch reference
(im2col and a matrix product).  Products of bfloat16 values are exact in FP32,
so a sum of K products in FP32 is off by at most (K - 1) 2^-24 of the sum of
their magnitudes, whatever the order; the bound is evaluated per output from
the same reference with absolute values, with K + 2 terms for the bias and
the final rounding.  Stored bfloat16 outputs are the FP32 ones rounded.
"""
import pytest
import torch

from gpu_util import announce

pytestmark = pytest.mark.gpu


def _rand(g, *shape):
    return torch.randn(*shape, device="cuda", generator=g).to(torch.bfloat16)


def _columns(x):
    """Patches [pixels][9 C] (tap-major) of x [B][H][W][C], 64 bits."""
    B, H, W, C = x.shape
    c = torch.nn.functional.unfold(x.double().permute(0, 3, 1, 2), 3, padding=1, stride=2)
    return c.view(B, C, 9, -1).permute(0, 3, 2, 1).reshape(-1, 9 * C)


def _check(got32, got16, ref, mag, terms, what):
    bound = (terms + 2) * 2.0 ** -24 * mag
    err = (got32.double() - ref).abs()
    announce(f"  {what}: max |error| / bound = {float((err / bound.clamp_min(1e-300)).max()):.3f}")
    assert bool((err <= bound).all())
    if got16 is not None:
        assert torch.equal(got16, got32.to(torch.bfloat16))


# (B, H, W, Cin, Cout): rows and columns around every tile the launch chooses
@pytest.mark.parametrize("B,H,W,Cin,Cout", [
    (1, 2, 2, 32, 8), (1, 6, 4, 64, 40), (3, 10, 14, 32, 72), (2, 8, 8, 96, 136),
    (130, 32, 32, 32, 64), (131, 32, 32, 32, 72), (70, 32, 32, 64, 136), (257, 16, 32, 32, 128),
    (33, 64, 64, 32, 64), (5, 12, 12, 40, 24),
])
def test_conv_forward_tiles(gpu_lib, B, H, W, Cin, Cout):
    announce(f"conv forward B={B} {H}x{W} {Cin}->{Cout}")
    g = torch.Generator(device="cuda").manual_seed(5)
    x, w = _rand(g, B, H, W, Cin), _rand(g, Cout, 3, 3, Cin)
    bias = torch.randn(Cout, device="cuda", generator=g)
    y, y32 = gpu_lib.conv_forward(x, w, bias, relu=False, want_f32=True)
    cols, wm = _columns(x), w.double().reshape(Cout, -1)
    ref = cols @ wm.t() + bias.double()
    mag = cols.abs() @ wm.abs().t() + bias.double().abs()
    _check(y32.reshape(-1, Cout), y.reshape(-1, Cout), ref, mag, 9 * Cin, "forward")


# (B, H, W, Cin, Cout) of the layer whose data gradient is taken
@pytest.mark.parametrize("B,H,W,Cin,Cout", [
    (1, 2, 2, 8, 32), (1, 6, 4, 40, 64), (3, 10, 14, 72, 32), (2, 8, 8, 136, 96),
    (9, 64, 64, 32, 64), (33, 32, 32, 64, 32), (34, 32, 32, 72, 64), (17, 64, 64, 128, 32),
    (4, 12, 12, 24, 40),
])
@pytest.mark.parametrize("masked", [False, True])
def test_conv_dgrad_tiles(gpu_lib, B, H, W, Cin, Cout, masked):
    announce(f"conv dgrad B={B} {H}x{W} {Cin}->{Cout} masked={masked}")
    g = torch.Generator(device="cuda").manual_seed(6)
    dy, w = _rand(g, B, H // 2, W // 2, Cout), _rand(g, Cout, 3, 3, Cin)
    act = _rand(g, B, H, W, Cin) if masked else None
    dx, dx32 = gpu_lib.conv_dgrad(dy, w.permute(3, 1, 2, 0).contiguous(), act, want_f32=True)

    def adjoint(d, wt):
        cols = (d.reshape(-1, Cout) @ wt.reshape(Cout, -1)).view(B, -1, 9, Cin)
        cols = cols.permute(0, 3, 2, 1).reshape(B, 9 * Cin, -1)
        return torch.nn.functional.fold(cols, (H, W), 3, padding=1, stride=2).permute(0, 2, 3, 1)

    ref, mag = adjoint(dy.double(), w.double()), adjoint(dy.double().abs(), w.double().abs())
    if masked:
        ref = ref * (act > 0)
    _check(dx32, dx, ref, mag, 9 * Cout, "dgrad")


# one split and several, remainders of the 32-pixel steps, tiles of 64 and 128
# output channels, ragged (tap, channel) columns; the first layer's row kernel
# (32 channels, rows of whole steps) and its general one
@pytest.mark.parametrize("B,H,W,Cin,Cout", [
    (1, 2, 2, 8, 8), (1, 6, 10, 24, 72), (3, 10, 14, 40, 64), (2, 8, 8, 96, 136),
    (9, 48, 48, 32, 64), (33, 32, 32, 64, 128), (5, 66, 34, 16, 200), (7, 64, 64, 128, 256),
    (1, 64, 64, 1, 32), (5, 64, 128, 1, 32), (70, 64, 64, 1, 32), (3, 32, 32, 1, 32), (2, 64, 64, 1, 24),
])
def test_conv_wgrad_tiles(gpu_lib, B, H, W, Cin, Cout):
    announce(f"conv wgrad B={B} {H}x{W} {Cin}->{Cout}")
    g = torch.Generator(device="cuda").manual_seed(7)
    x, dy = _rand(g, B, H, W, Cin), _rand(g, B, H // 2, W // 2, Cout)
    dw = gpu_lib.conv_wgrad(dy, x)
    d, cols = dy.double().reshape(-1, Cout), _columns(x)
    _check(dw.reshape(Cout, -1), None, d.t() @ cols, d.abs().t() @ cols.abs(), d.shape[0], "wgrad")
