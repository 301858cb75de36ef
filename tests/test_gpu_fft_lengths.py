"""FFT passes at every supported length against 64-bit torch (GPU).

A transform of length D in FP32 has a relative 2-norm error of at most
5 log2(D) 2^-24 (each butterfly level adds a few roundings); filtering an
image takes four of them and a multiplier of magnitude at most 1 accurate to
about 2^-22, so the bound is (20 log2(D) + 4) 2^-24 of the image's 2-norm.
"""
import math

import numpy as np
import pytest
import torch

from oracle import ctf as o_ctf
from oracle import objective as o_obj
from oracle import trainer as o_trainer
from paper_2508_04929_amd import binding, inputs

from gpu_util import announce, ctf_arg, dev, host, mixture_args

pytestmark = pytest.mark.gpu
PIXEL = float(np.float32(1.3))  # the library takes it in FP32: both sides get the same value
LENGTHS = sorted(2 ** a * 3 ** b for a in range(1, 10) for b in range(6) if 2 ** a * 3 ** b <= 512)


def _bound(D):
    return (20 * math.log2(D) + 4) * 2.0 ** -24


def _check(got, ref, scale, D, what):
    err = np.sqrt(((host(got) - ref) ** 2).sum((1, 2)))
    announce(f"  {what} D={D}: max error / bound = {np.max(err / (_bound(D) * scale)):.3f}")
    assert np.all(err <= _bound(D) * scale)


@pytest.mark.parametrize("D", LENGTHS)
@pytest.mark.parametrize("B", [1, 33])
def test_filter_and_shift(gpu_lib, D, B):
    rng = np.random.default_rng(D)
    Y = rng.standard_normal((B, D, D)).astype(np.float32)
    norm = np.sqrt((Y.astype(np.float64) ** 2).sum((1, 2)))
    v = inputs.views(rng, B, D, PIXEL)
    v.defocus_v = v.defocus_v - 300
    v.astig = rng.uniform(0, 3, B).astype(np.float32)
    H = o_ctf.ctf_grid_for(v)
    _check(gpu_lib.ctf_filter(dev(Y), ctf_arg(v), PIXEL), o_ctf.apply_ctf(Y.astype(np.float64), H), norm, D,
           "filter")
    t = rng.uniform(-3, 3, (B, 2)).astype(np.float32)
    _check(gpu_lib.fourier_shift(dev(Y), dev(t), PIXEL, direction=-1),
           o_trainer.fourier_shift(Y.astype(np.float64), -t.astype(np.float64), PIXEL), norm, D, "shift")


@pytest.mark.parametrize("D", LENGTHS)
def test_loss_and_adjoint_images(gpu_lib, D):
    """The fused loss rows: X, the loss and, through one wide Gaussian per
    corner, the gradient against the oracle."""
    rng = np.random.default_rng(1000 + D)
    g = inputs.mixture_anisotropic(rng, 4, 0.2 * D, scale_mu=np.log(1.2), scale_sd=0.05)
    v = inputs.views(rng, 2, D, 1.0)
    Y = rng.standard_normal((2, D, D)).astype(np.float32)
    loss, grads, X = gpu_lib.loss_and_grad(**mixture_args(g), rot=dev(v.rot), shift=dev(v.shift), D=D,
                                           pixel=1.0, observed=dev(Y), ctf=ctf_arg(v), want_images=True)
    ref = o_obj.loss_and_grad(g, v, Y, q_cut=2 * np.log(1e6))
    np.testing.assert_allclose(host(X), ref["X"], atol=1e-4 * np.abs(ref["X"]).max())
    assert abs(float(loss[-1]) - ref["loss"]) <= 1e-4 * abs(ref["loss"])
    for k in ("means", "log_scales", "amps"):
        np.testing.assert_allclose(host(grads[k]), ref["grads"][k], atol=1e-3 * np.abs(ref["grads"][k]).max())
