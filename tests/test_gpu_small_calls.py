"""Calls of few Gaussian-image pairs: smaller tiles and work items, and four
lanes to a record in both splat kernels.  Sizes on both sides of each line (32768
and 524288 pairs, 256 default tiles, a halo above the default), ragged images, records
wider than the halo, and options given one by one, against the FP64 oracle.

Images within 1e-4 normwise, gradients within 1e-3, the renderer's bars: the
record sums are the same FP32 terms in another order."""
import numpy as np
import pytest

from oracle import ctf as o_ctf
from oracle import model as o_model
from oracle import objective as o_obj
from paper_2508_04929_amd import binding, inputs

from gpu_util import announce, ctf_arg, dev, host, mixture_args, normwise, per_image_normwise, view_args

pytestmark = pytest.mark.gpu

Q_MATCHED = 2.0 * np.log(1e6)


@pytest.mark.parametrize("n,b,D,sd,opt", [
    (1, 1, 16, 1.0, {}),
    (3, 2, 33, 1.0, {}),                    # one row and column past a 32 tile
    (65, 1, 64, 0.8, {}),                   # one record past a work item
    (300, 3, 70, 5.0, {}),                  # records wider than the halo beside narrow ones
    (200, 2, 48, 1.5, {"halo": 20}),        # halo above the default: default tile
    (200, 2, 48, 1.5, {"halo": 8}),
    (200, 2, 48, 1.5, {"tile": 48}),
    (200, 2, 48, 1.5, {"budget": 100}),
    (200, 2, 48, 1.5, {"lane_order": 1}),
    (200, 2, 48, 1.5, {"lane_order": 2}),
    (20, 64, 128, 1.5, {}),                 # 256 default tiles
    (20, 65, 128, 1.5, {}),                 # 260
    (4096, 8, 32, 0.7, {}),                 # 32768 pairs
    (4097, 8, 32, 0.7, {}),
    (4096, 128, 24, 0.7, {}),               # 524288 pairs: four lanes
    (4097, 128, 24, 0.7, {}),               # more: one
])
def test_small_calls_match_the_oracle(gpu_lib, n, b, D, sd, opt):
    rng = np.random.default_rng(n + b + D)
    g = inputs.mixture_anisotropic(rng, n, 0.4 * D, scale_mu=np.log(sd), scale_sd=0.6)
    v = inputs.views(rng, b, D, 1.0, shift_px_sd=1.0)
    dX = rng.standard_normal((b, D, D)).astype(np.float32)
    o = binding.Options(**opt)
    announce(f"small call N={n} B={b} D={D} {opt}")
    Q = host(gpu_lib.render(**mixture_args(g), **view_args(v), options=o))
    ref = o_model.render_pre_ctf(g.means, g.log_scales, g.quats, g.amps, v.rot, v.shift, v.D,
                                 v.pixel, Q_MATCHED)
    assert per_image_normwise(Q, ref) <= 1e-4
    got = gpu_lib.render_backward(**mixture_args(g), **view_args(v), d_images=dev(dX), options=o)
    want = o_obj.backward_from_image_grad(g, v, dX, q_cut=Q_MATCHED)
    for k in ("means", "log_scales", "quats", "amps"):
        assert normwise(host(got[k]), want[k]) <= 1e-3, k


def test_limited_workspace_falls_back_to_the_default_tile(monkeypatch):
    """1000 Gaussians in one 64 x 64 image need about 0.44 MB with the small
    tile and 0.30 MB with the default one: under a limit of 0.40 MB the call
    still runs, with the default tile's bits."""
    rng = np.random.default_rng(3)
    g = inputs.mixture_anisotropic(rng, 1000, 25.0)
    v = inputs.views(rng, 1, 64, 1.0)
    monkeypatch.setenv("CS_WORKSPACE_MAX", "400000")
    lib = binding.Library(binding.load_library())
    announce("small call under a workspace limit")
    auto = host(lib.render(**mixture_args(g), **view_args(v)))
    tile = host(lib.render(**mixture_args(g), **view_args(v),
                           options=binding.Options(tile=64, halo=16, budget=256)))
    assert np.array_equal(auto, tile)
    monkeypatch.delenv("CS_WORKSPACE_MAX")
    free = host(binding.Library(binding.load_library()).render(**mixture_args(g), **view_args(v)))
    assert per_image_normwise(free, auto) <= 1e-5


@pytest.mark.parametrize("n,b,D", [
    (4096, 6, 108),    # 16 Gaussian blocks: a thread scans a bin's counts
    (4097, 6, 108),    # 17: a wave does
    (1000, 16, 128),   # 272 bins of 4 blocks: a thread
    (4500, 7, 216),    # 350 bins of 18 blocks: a kernel of its own
    (17000, 1, 64),    # 67 blocks: a wave in two steps
    (4096, 128, 24),   # 524288 pairs: Gaussians built while counting
    (4097, 128, 24),   # more: beforehand
    (50, 32, 36),      # 32 images: losses in one launch
    (50, 33, 36),      # 33: in two
])
def test_binning_and_loss_lines_match_the_oracle(gpu_lib, n, b, D):
    """Images within 1e-4 normwise and losses within 1e-4, the renderer's bars."""
    rng = np.random.default_rng(n + b + D)
    g = inputs.mixture_anisotropic(rng, n, 0.4 * D, scale_mu=np.log(0.7))
    v = inputs.views(rng, b, D, 1.0)
    announce(f"binning and loss N={n} B={b} D={D}")
    ref = o_ctf.apply_ctf(o_model.render_pre_ctf(g.means, g.log_scales, g.quats, g.amps, v.rot, v.shift, v.D,
                                                 v.pixel, Q_MATCHED), o_ctf.ctf_grid_for(v))
    Y = (0.5 * ref + ref.std() * rng.standard_normal(ref.shape)).astype(np.float32)
    loss, _, X = gpu_lib.loss_and_grad(**mixture_args(g), **view_args(v), observed=dev(Y), ctf=ctf_arg(v),
                                       want_grads=False, want_images=True)
    assert per_image_normwise(host(X), ref) <= 1e-4
    per, _ = o_obj.loss_from_images(ref, Y, "sum")
    np.testing.assert_allclose(host(loss)[:-1], per, rtol=1e-4)
    np.testing.assert_allclose(host(loss)[-1], per.sum(), rtol=1e-4)


@pytest.mark.parametrize("n,b,D", [(4096, 128, 24), (4097, 128, 24), (70001, 8, 64)])
def test_automatic_lane_order_keeps_the_bits(gpu_lib, n, b, D):
    """Untuned calls above 524288 pairs sort their records; with a tile given the
    order is the caller's (here the list's).  Both sum the same terms."""
    rng = np.random.default_rng(n)
    g = inputs.mixture_anisotropic(rng, n, 0.4 * D, scale_mu=np.log(0.8), scale_sd=0.5)
    v = inputs.views(rng, b, D, 1.0)
    Y = dev(rng.standard_normal((b, D, D)).astype(np.float32))
    announce(f"automatic lane order N={n} B={b} D={D}")
    kw = dict(**mixture_args(g), **view_args(v), observed=Y, want_images=True)
    auto = gpu_lib.loss_and_grad(**kw)
    listed = gpu_lib.loss_and_grad(**kw, options=binding.Options(tile=64))
    assert np.array_equal(host(auto[2]), host(listed[2]))
    for k in auto[1]:
        assert np.array_equal(host(auto[1][k]), host(listed[1][k])), k
