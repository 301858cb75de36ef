"""Grid-search scores at the edges of the score GEMM's tiles (GPU).

The search runs whole rounds of 256 x 256 tiles and the rest as 128 x 128
parts; refinement with explicit candidates computes the same scores from the
same bfloat16 operands with another kernel.  Both accumulate n = D^2 +
D (D / 2 + 1) products in FP32, so with |H| <= 1 they differ by at most
2 n 2^-24 (||Y|| + ||Q||)^2 per score.
"""
import numpy as np
import pytest
import torch

from paper_2508_04929_amd import inputs

from gpu_util import announce, ctf_arg, dev, host, mixture_args

pytestmark = pytest.mark.gpu


# (particles, rotations, shift radius): rows = particles (2r + 1)^2
@pytest.mark.parametrize("P,K,r", [
    (1, 1, 0), (1, 129, 1), (28, 256, 1), (29, 257, 1),  # 252 and 261 rows: one tile, two
    (256, 4096, 0), (300, 6000, 1),                       # 16 tiles; 11 x 24 = 264: one round + 8
    (5, 6000, 2), (455, 4097, 1),                         # 24 tiles; 16 x 17 = 272: one round + 16
])
def test_search_scores_equal_refinement_scores(gpu_lib, P, K, r):
    announce(f"search vs refinement scores, P={P}, K={K}, r={r}")
    rng = np.random.default_rng(77)
    D, pixel = 16, 1.5
    g = inputs.mixture_anisotropic(rng, 60, 4.0, scale_mu=np.log(1.0), scale_sd=0.1)
    v = inputs.views(rng, P, D, pixel)
    G = inputs.haar_rotations(rng, K).astype(np.float32)
    Y = rng.standard_normal((P, D, D)).astype(np.float32)
    Q = gpu_lib.render(**mixture_args(g), rot=dev(G), shift=None, D=D, pixel=pixel)
    bank = gpu_lib.pose_bank(**mixture_args(g), rot=dev(G), n_psi=0, D=D, pixel=pixel)
    batch = gpu_lib.pose_batch(D, pixel, P, r)
    batch.load(dev(Y), ctf_arg(v))
    out = batch.search(bank, want_scores=True)
    cand = np.unique(np.concatenate([np.arange(K)[:3], np.arange(K)[-3:], rng.integers(0, K, 20),
                                     np.clip([127, 128, 255, 256], 0, K - 1)])).astype(np.int32)
    ref = batch.refine(bank, cand=torch.from_numpy(np.tile(cand, (P, 1))).cuda(), want_scores=True)
    torch.cuda.synchronize()
    scores = host(out["scores"])
    q_norm = np.sqrt((host(Q) ** 2).sum((1, 2)).max())
    y_norm = np.sqrt((Y.astype(np.float64) ** 2).sum((1, 2)))
    bound = (D * D + D * (D // 2 + 1)) * 2.0 ** -23 * (y_norm + q_norm) ** 2
    err = np.abs(scores[:, cand] - host(ref["scores"])).max((1, 2))
    announce(f"  max |difference| / bound = {np.max(err / bound):.3f}")
    assert np.all(err <= bound)
    # the reported minimum is the first of the smallest reported scores
    flat = scores.reshape(P, -1)
    S = (2 * r + 1) ** 2
    best = flat.argmin(1)
    np.testing.assert_array_equal(out["rot_idx"].cpu().numpy(), best // S)
    np.testing.assert_array_equal(out["shift_idx"].cpu().numpy(), best % S)
    np.testing.assert_array_equal(host(out["score"]), flat.min(1))
    bank.close()
    batch.close()
