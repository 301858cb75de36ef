"""Rounding of long FP32 sums on data that rounds the same way at every step
(GPU): the squared residuals of a row pair, and the adjoint's moments of a record
wider than its image."""
import numpy as np
import pytest

from paper_2508_04929_amd import inputs

from gpu_util import announce, ctf_arg, dev, host, mixture_args, view_args

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D", [32, 256, 486])
def test_loss_of_constant_residuals(gpu_lib, D):
    """Zero images against a constant: a loss may be off by the rounding of a row
    pair's sum and of the result, 2^-24 each."""
    c = np.float32(1.896690070210632)
    rng = np.random.default_rng(D)
    g = inputs.mixture_anisotropic(rng, 3, 0.2 * D)
    g.amps[:] = 0.0
    v = inputs.views(rng, 2, D, 1.0)
    announce(f"loss of a constant, D={D}")
    loss, _, X = gpu_lib.loss_and_grad(**mixture_args(g), **view_args(v), ctf=ctf_arg(v),
                                       observed=dev(np.full((2, D, D), c)), want_images=True)
    assert not host(X).any()
    ref = D * D * float(c) ** 2
    assert np.abs(host(loss)[:2] - ref).max() <= 1.001 * 2.0 ** -23 * ref


@pytest.mark.parametrize("D,n", [(64, 1), (65, 1), (512, 1), (512, 520)])
def test_moment_of_a_record_over_the_whole_image(gpu_lib, D, n):
    """exp is 1 at every pixel, so dL/dA is the sum of a constant image over it,
    times the record's norm.  A lane of 64 adds at most D^2 / 64 values in runs of
    eight, the lanes meet in a tree, and the chain to dL/dA and the norm add some 20
    roundings: (8 + D^2 / 512 + 7 + 6 + 20) 2^-24."""
    c = np.float32(1.0277099609375)
    rng = np.random.default_rng(D)
    g = inputs.mixture_anisotropic(rng, n, 0.1 * D)
    g.log_scales[:] = np.float32(np.log(1e8))
    g.amps[:] = 1.0
    v = inputs.views(rng, 1, D, 1.0)
    announce(f"moment of a constant, D={D}, {n} records")
    got = gpu_lib.render_backward(**mixture_args(g), **view_args(v),
                                  d_images=dev(np.full((1, D, D), c)))["amps"]
    sigma = float(np.exp(np.float64(g.log_scales[0, 0])))
    ref = float(c) * D * D / (2.0 * np.pi * sigma ** 2)
    assert np.abs(host(got) - ref).max() <= (41 + D * D / 512) * 2.0 ** -24 * ref
