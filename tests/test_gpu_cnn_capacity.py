"""Training batches smaller than a network's capacity.

The partial sums of the weight gradients are allocated once for the capacity,
so what a batch needs may not exceed what the capacity was given."""
import ctypes
import os

import pytest
import torch

from paper_2508_04929_amd import binding

from gpu_util import announce

CHANNELS = (1, 32, 64, 128, 256, 256, 256)


@pytest.mark.skipif(not os.path.exists(binding.LIB_PATH), reason="libcryosplat.so not built")
@pytest.mark.parametrize("D,cap", [(64, 600), (128, 300), (192, 140), (256, 140), (512, 40)])
def test_partials_never_shrink_with_the_batch(D, cap):
    """Sizes of the partial sums of every layer, host code: none is larger for a
    smaller batch."""
    lib = binding.load_library()
    conv, lin = lib._ZN2cs15conv_wgrad_partEiiiiib, lib._ZN2cs14lin_wgrad_partEiii
    conv.restype = lin.restype = ctypes.c_size_t
    side = D
    for ci, co in zip(CHANNELS, CHANNELS[1:]):
        n = [conv(b, side, side, ci, co, True) for b in range(1, cap + 1)]
        assert all(a <= b for a, b in zip(n, n[1:])), (side, ci, co)
        side //= 2
    for i, o in ((side * side * 256, 256), (256, 8)):
        n = [lin(b, i, o) for b in range(1, cap + 1)]
        assert all(a <= b for a, b in zip(n, n[1:])), (i, o)


@pytest.mark.gpu
@pytest.mark.parametrize("D,cap,batches", [(128, 256, (255, 200, 85)), (256, 64, (33,)), (64, 512, (500,))])
def test_gradients_do_not_depend_on_the_capacity(gpu_lib, D, cap, batches):
    """The same bits as from a network made for exactly that batch."""
    g = torch.Generator(device="cuda").manual_seed(D)
    x = torch.randn(cap, D, D, device="cuda", generator=g)
    rot = torch.linalg.qr(torch.randn(cap, 3, 3, device="cuda", generator=g))[0].contiguous()
    shift = torch.randn(cap, 2, device="cuda", generator=g)
    net = gpu_lib.network(D, max_batch=cap, seed=5)
    for b in batches:
        announce(f"network D={D}: {b} of {cap}")
        own = gpu_lib.network(D, max_batch=b, seed=5)
        a = [n.train_step(x[:b], rot[:b], shift[:b], update=False, want_grads=True) for n in (net, own)]
        assert torch.equal(a[0][0], a[1][0]) and torch.equal(a[0][1], a[1][1])
        own.close()
    net.close()
