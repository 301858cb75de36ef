"""Rounding of long sums on data that rounds the same way at every step (GPU):
the squared residuals of a row pair."""
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
