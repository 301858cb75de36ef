"""Voxelisation with more (brick, Gaussian) pairs than its 32-bit lists hold (GPU):
refused, whatever the pairs come to modulo 2^32, and the next call is sound."""
import numpy as np
import pytest

from oracle import volume as o_vol
from paper_2508_04929_amd import binding, inputs

from gpu_util import announce, host, mixture_args, normwise

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,n", [
    (512, 8192),     # 2^31 pairs: negative in 32 bits
    (512, 16384),    # 2^32: zero
    (256, 150000),   # 4.9e9: 6.2e8
])
def test_too_many_pairs_are_refused(gpu_lib, D, n):
    announce(f"{n} Gaussians over a volume of {D}^3")
    rng = np.random.default_rng(n)
    g = inputs.mixture_anisotropic(rng, n, 10.0, scale_mu=np.log(10.0 * D), scale_sd=0.0)
    with pytest.raises(binding.CryoSplatError, match="too many"):
        gpu_lib.voxelize(**mixture_args(g), D=D, pixel=1.0)
    s = inputs.mixture_anisotropic(rng, 50, 8.0)
    assert normwise(host(gpu_lib.voxelize(**mixture_args(s), D=24, pixel=1.0)),
                    o_vol.voxelize(s, 24, 1.0, q_cut=2.0 * np.log(1e6))) <= 1e-4
