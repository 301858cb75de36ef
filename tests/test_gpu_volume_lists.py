"""Voxel lists in two levels (cells of 2^3 bricks, 4^3 above 256^3) and shell
sums by symmetric quadruples: sizes at the edges of cells and bricks, Gaussians
from below a voxel to the whole volume, signed weights, empty volumes.

Volumes within 1e-4 normwise, the voxelisation's bar; FSC within 1e-4 absolute
of the correlation in FP64 (FP32 transforms: some 1e-6 per coefficient)."""
import numpy as np
import pytest
import torch

from oracle import volume as o_vol
from paper_2508_04929_amd import inputs

from gpu_util import announce, dev, host, mixture_args, normwise

pytestmark = pytest.mark.gpu

Q_MATCHED = 2.0 * np.log(1e6)


@pytest.mark.parametrize("n,D,sd,signed", [
    (1, 8, 1.0, False),       # one brick
    (700, 24, 0.8, True),     # three bricks a side: a cell and a half
    (513, 40, 6.0, True),     # boxes of many cells; one Gaussian past a block's pass
    (3000, 16, 0.2, False),   # one cell, six passes, sub-voxel Gaussians
])
def test_voxel_lists_match_the_oracle(gpu_lib, n, D, sd, signed):
    rng = np.random.default_rng(n + D)
    g = inputs.mixture_anisotropic(rng, n, 0.6 * D, scale_mu=np.log(sd), scale_sd=0.5)
    if signed:
        g.amps[::3] *= -1.0
    announce(f"voxel lists N={n} D={D} sd={sd}")
    V = gpu_lib.voxelize(**mixture_args(g), D=D, pixel=1.0)
    assert normwise(host(V), o_vol.voxelize(g, D, 1.0, q_cut=Q_MATCHED)) <= 1e-4


@pytest.mark.parametrize("D", [256, 264])
def test_cells_of_both_sizes_at_sampled_voxels(gpu_lib, D):
    rng = np.random.default_rng(D)
    g = inputs.mixture_anisotropic(rng, 2000, 0.49 * D, scale_mu=np.log(2.0), scale_sd=0.6)
    announce(f"voxel lists D={D}, sampled")
    V = host(gpu_lib.voxelize(**mixture_args(g), D=D, pixel=1.0))
    near = np.rint(g.means[:400, ::-1] + rng.uniform(-4, 4, (400, 3))).astype(int) + D // 2
    idx = np.concatenate([np.clip(near, 0, D - 1), rng.integers(0, D, (400, 3))])
    ref = o_vol.density_at(g, o_vol.voxel_points(D, 1.0, idx), q_cut=Q_MATCHED)
    assert np.abs(V[idx[:, 0], idx[:, 1], idx[:, 2]] - ref).max() <= 1e-4 * V.max()


@pytest.mark.parametrize("D", [2, 6, 24, 54])
def test_shell_sums_match_numpy(gpu_lib, D):
    rng = np.random.default_rng(D)
    a = rng.standard_normal((D, D, D)).astype(np.float32)
    b = (a + 0.7 * rng.standard_normal((D, D, D))).astype(np.float32)
    announce(f"FSC D={D}")
    assert np.abs(host(gpu_lib.fsc(dev(a), dev(b))) - o_vol.fsc(a, b)).max() <= 1e-4
