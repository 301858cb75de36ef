"""Images of wide and narrow records where the threads that share a group of pixels
change (1, 4, 16, 64) and where its tiles are cut into more blocks (GPU).  Images
within 1e-4 normwise of the FP64 oracle, the renderer's bar."""
import numpy as np
import pytest

from oracle import model as o_model
from paper_2508_04929_amd import inputs

from gpu_util import announce, dev, host, mixture_args, per_image_normwise, view_args

pytestmark = pytest.mark.gpu

Q_MATCHED = 2.0 * np.log(1e6)


@pytest.mark.parametrize("n,b,D", [
    (4095, 1, 16), (4096, 1, 16), (5000, 4, 19), (16384, 1, 64), (16384, 2, 63),  # 16 and 64 threads
    (255, 1, 16), (256, 1, 17), (1023, 1, 64), (1024, 1, 64), (2560, 4, 100),     # 4 and 16
    (2560, 5, 100), (5120, 4, 143), (5184, 4, 144),
    (1056, 32, 65), (1024, 32, 65), (1023, 32, 65),   # 4, 1 in more blocks, 1
])
def test_shared_pixel_groups_match_the_oracle(gpu_lib, n, b, D):
    announce(f"{n} records, some wide, in {b} images of {D}^2")
    rng = np.random.default_rng(n + b + D)
    g = inputs.mixture_anisotropic(rng, n, 0.4 * D, scale_mu=np.log(2.0), scale_sd=0.8)
    v = inputs.views(rng, b, D, 1.0, shift_px_sd=1.0)
    got = gpu_lib.render(**mixture_args(g), **view_args(v))
    want = o_model.render_pre_ctf(g.means, g.log_scales, g.quats, g.amps, v.rot, v.shift, v.D, v.pixel, Q_MATCHED)
    assert per_image_normwise(host(got), want) <= 1e-4
