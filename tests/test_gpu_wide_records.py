"""Adjoint of records wider than the halo, few and many to an image: a block to a
record up to three times the number of blocks that share an image (512 over the
images, at least 4), a wave beyond (GPU).  Gradients within 1e-3 normwise of the FP64 oracle,
the renderer's bar."""
import numpy as np
import pytest

from oracle import objective as o_obj
from paper_2508_04929_amd import inputs

from gpu_util import announce, dev, host, mixture_args, normwise, view_args

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,b,D", [(1, 1, 33), (2, 1, 200), (511, 1, 24), (513, 1, 24), (1536, 1, 16),
                                   (1537, 1, 16), (3, 128, 40), (4, 128, 40), (5, 128, 40), (12, 130, 17),
                                   (13, 130, 17)])
def test_wide_records_match_the_oracle(gpu_lib, n, b, D):
    announce(f"{n} wide records in each of {b} images of {D}^2")
    rng = np.random.default_rng(n + b)
    g = inputs.mixture_anisotropic(rng, n, 0.4 * D, scale_mu=np.log(12.0), scale_sd=0.3)
    v = inputs.views(rng, b, D, 1.0, shift_px_sd=1.0)
    dX = rng.standard_normal((b, D, D)).astype(np.float32)
    got = gpu_lib.render_backward(**mixture_args(g), **view_args(v), d_images=dev(dX))
    want = o_obj.backward_from_image_grad(g, v, dX, q_cut=2.0 * np.log(1e6))
    for k in ("means", "log_scales", "quats", "amps"):
        assert normwise(host(got[k]), want[k]) <= 1e-3, k
