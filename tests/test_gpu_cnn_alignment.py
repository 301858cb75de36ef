"""Single-layer calls on views that start off a 16-byte boundary (GPU).

Forward and data gradient add the same products in the same order as on aligned
operands, so the bits are the same; the weight gradient splits its pixels in
another way and is within (pixels) 2^-24 of the sum of magnitudes of the aligned
one, twice."""
import pytest
import torch

from gpu_util import announce

pytestmark = pytest.mark.gpu


def _off(t, k):
    """A copy of t that starts k elements past an allocation."""
    buf = torch.empty(t.numel() + 16, device=t.device, dtype=t.dtype)
    v = buf[k:k + t.numel()].view(t.shape)
    v.copy_(t)
    assert v.data_ptr() % 16 == 2 * k % 16
    return v


@pytest.mark.parametrize("k", [1, 2, 4])
@pytest.mark.parametrize("B,H,W,Cin,Cout", [(2, 8, 6, 32, 32), (3, 34, 34, 64, 72), (2, 10, 12, 40, 24),
                                            (40, 32, 32, 32, 128), (2, 64, 64, 1, 32)])
def test_offset_views(gpu_lib, B, H, W, Cin, Cout, k):
    announce(f"{Cin}->{Cout} of {B} {H}x{W}, {2 * k} bytes off")
    g = torch.Generator(device="cuda").manual_seed(9)

    def rand(*shape):
        return torch.randn(*shape, device="cuda", generator=g).to(torch.bfloat16)

    x, w, dy = rand(B, H, W, Cin), rand(Cout, 3, 3, Cin), rand(B, H // 2, W // 2, Cout)
    bias = torch.randn(Cout, device="cuda", generator=g)
    a = gpu_lib.conv_forward(x, w, bias, want_f32=True)
    for args in ((_off(x, k), w), (x, _off(w, k))):
        b = gpu_lib.conv_forward(*args, bias, want_f32=True)
        assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])
    if Cin > 1:
        wt = w.permute(3, 1, 2, 0).contiguous()
        a = gpu_lib.conv_dgrad(dy, wt, x, want_f32=True)
        for args in ((_off(dy, k), wt, x), (dy, _off(wt, k), x), (dy, wt, _off(x, k))):
            b = gpu_lib.conv_dgrad(*args, want_f32=True)
            assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])
    a, mag = gpu_lib.conv_wgrad(dy, x), gpu_lib.conv_wgrad(dy.abs(), x.abs())
    bound = 2.0 * B * (H // 2) * (W // 2) * 2.0 ** -24 * mag * 1.001
    for args in ((_off(dy, k), x), (dy, _off(x, k))):
        assert bool(((gpu_lib.conv_wgrad(*args) - a).abs() <= bound).all())
