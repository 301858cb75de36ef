"""Fourier shift of an image alone and in a batch (GPU): four columns per block
where the blocks of 16 (8 above 256 points) would not fill the chip, the same bits
either way."""
import pytest
import torch

from gpu_util import announce

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,B", [(6, 300), (24, 128), (128, 52), (256, 29), (486, 9)])
def test_a_batch_shifts_as_its_images_do(gpu_lib, D, B):
    announce(f"shift of {B} images of {D}^2")
    g = torch.Generator(device="cuda").manual_seed(D)
    Y = torch.randn(B, D, D, device="cuda", generator=g)
    t = 6.0 * torch.rand(B, 2, device="cuda", generator=g) - 3.0
    whole = gpu_lib.fourier_shift(Y, t, 1.25)
    for b in (0, B // 2, B - 1):
        one = gpu_lib.fourier_shift(Y[b:b + 1].contiguous(), t[b:b + 1].contiguous(), 1.25)
        assert torch.equal(one[0], whole[b])
