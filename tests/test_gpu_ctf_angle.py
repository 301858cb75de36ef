"""Without astigmatism (equal defoci) the azimuth does not enter the CTF, so a
missing one, stored as NaN or infinity, changes no bit (GPU)."""
import numpy as np
import pytest
import torch

from paper_2508_04929_amd import inputs

from gpu_util import announce, ctf_arg, dev, mixture_args, view_args

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D", [48, 128])
@pytest.mark.parametrize("angle", [float("nan"), float("inf")])
def test_azimuth_of_equal_defoci_is_not_read(gpu_lib, D, angle):
    announce(f"CTF azimuth {angle}, D={D}")
    rng = np.random.default_rng(D)
    g = inputs.mixture_anisotropic(rng, 200, 0.3 * D)
    v = inputs.views(rng, 4, D, 1.5)
    v.defocus_v = v.defocus_u.copy()
    Y = dev(rng.standard_normal((4, D, D)).astype(np.float32))

    def results(a):
        v.astig = np.full(4, a, dtype=np.float32)
        c, kw = ctf_arg(v), dict(**mixture_args(g), **view_args(v))
        loss, grads, X = gpu_lib.loss_and_grad(**kw, ctf=c, observed=Y, want_images=True)
        back = gpu_lib.render_backward(**kw, ctf=c, d_images=Y)
        z = torch.empty_like(Y)
        batch = gpu_lib.pose_batch(D, 1.5, 4, 1)
        batch.load(Y, c, filtered=z)
        torch.cuda.synchronize()
        batch.close()
        return [loss, X, gpu_lib.ctf_filter(Y, c, 1.5), z, *grads.values(), *back.values()]

    for a, b in zip(results(0.3), results(angle)):
        assert torch.equal(a, b)
