"""Weight gradient of a linear layer on its own: no bias gradient is asked for,
so no room for one may be either."""
import pytest
import torch

from gpu_util import announce

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,In,Out", [(32768, 8, 8200), (32768, 8, 8192)])
def test_many_rows_and_outputs(gpu_lib, B, In, Out):
    """1,024 chunks of 32 rows, whose column sums would pass 2^23 values.  Sums of
    B exact products in FP32: within B 2^-24 of the sum of magnitudes."""
    announce(f"linear wgrad B={B} {In}->{Out}")
    g = torch.Generator(device="cuda").manual_seed(8)
    x = torch.randn(B, In, device="cuda", generator=g).to(torch.bfloat16)
    dy = torch.randn(B, Out, device="cuda", generator=g).to(torch.bfloat16)
    dw = gpu_lib.linear_wgrad(dy, x)
    xd, d = x.double(), dy.double().t().contiguous()
    assert bool(((dw.double() - d @ xd).abs() <= B * 2.0 ** -24 * (d.abs() @ xd.abs())).all())
