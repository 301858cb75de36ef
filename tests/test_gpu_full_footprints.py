"""Records sorted by footprint where few, some and most are as tall as the image, which
the forward pass leaves in list order (GPU): both orders give the same bits."""
import numpy as np
import pytest

from paper_2508_04929_amd import binding, inputs

from gpu_util import announce, dev, host, mixture_args, view_args

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sd", [0.8, 1.5, 4.0])
@pytest.mark.parametrize("n,b,D", [(4097, 128, 16), (1025, 512, 23), (70001, 8, 32), (20000, 27, 40),
                                   (70001, 8, 97)])
def test_tall_records_keep_the_bits(gpu_lib, n, b, D, sd):
    announce(f"sorted and listed records N={n} B={b} D={D} sd={sd}")
    rng = np.random.default_rng(n)
    g = inputs.mixture_anisotropic(rng, n, 0.35 * D, scale_mu=np.log(sd), scale_sd=0.4)
    v = inputs.views(rng, b, D, 1.0)
    kw = dict(**mixture_args(g), **view_args(v), observed=dev(rng.standard_normal((b, D, D)).astype(np.float32)),
              want_images=True)
    a = gpu_lib.loss_and_grad(**kw)
    listed = gpu_lib.loss_and_grad(**kw, options=binding.Options(tile=64))
    assert np.array_equal(host(a[2]), host(listed[2]))
    for k in a[1]:
        assert np.array_equal(host(a[1][k]), host(listed[1][k])), k
