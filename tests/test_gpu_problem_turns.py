"""Blocks that pass through many problems of one launch (GPU): problems with a
handful of work items or none, more of them than a launch holds (16), against calls
of their own, bit for bit."""
import numpy as np
import pytest
import torch

from paper_2508_04929_amd import inputs

from gpu_util import announce, ctf_arg, dev, mixture_args, view_args

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("count", [2, 16, 35])
def test_short_and_empty_problems_in_turn(gpu_lib, count):
    announce(f"{count} short problems")
    probs = []
    for k in range(count):
        rng = np.random.default_rng(k)
        g = inputs.mixture_anisotropic(rng, 1 + 40 * (k % 5), 15.0)
        if k % 3 == 1:
            g.means[:] += np.float32(1e4)  # outside every image: no work items
        v = inputs.views(rng, 1 + k % 2, 48, 1.0)
        Y = dev(rng.standard_normal((v.rot.shape[0], 48, 48)).astype(np.float32))
        probs.append(gpu_lib.make_problem(**mixture_args(g), **view_args(v), observed=Y, ctf=ctf_arg(v),
                                          want_images=True))
    for _ in range(3):
        gpu_lib.loss_and_grad_multi(probs, use_graph=False)
    torch.cuda.synchronize()
    for pr in probs:
        loss, grads, X = gpu_lib.loss_and_grad(pr.means, pr.log_scales, pr.quats, pr.amps, pr.rot, pr.shift,
                                               pr.D, pr.pixel, pr.observed, ctf=pr.ctf, want_images=True)
        assert torch.equal(loss, pr.loss) and torch.equal(X, pr.images_out)
        for k in grads:
            assert torch.equal(grads[k], pr.grads[k]), k
