"""Grid-search scores of small batches (parts of 64 x 64 and 64 x 128 on a ring of
K steps) against the same particles in a batch of whole 256 x 256 tiles (GPU): both
add the same products in the same order, so the scores are the same bit for bit."""
import numpy as np
import pytest
import torch

from paper_2508_04929_amd import inputs

from gpu_util import announce, ctf_arg, dev, mixture_args

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,K,sizes", [
    (128, 1100, (1, 20, 110)),  # 5 and 10 tiles: 64 x 64; 55 tiles: 64 x 128; energies of 5 to 10
    (128, 9000, (1, 3)),        # 36 tiles: 64 x 128, and energies so against 128 x 128 parts of 72
    (96, 1100, (7,)),           # 144 K steps: no whole number of turns of the ring
])
def test_small_batches_score_as_large_ones(gpu_lib, D, K, sizes):
    rng = np.random.default_rng(D + K)
    P, r, pixel = 512, 2, 1.5
    g = inputs.mixture_anisotropic(rng, 200, 0.2 * D * pixel, scale_mu=np.log(2.0))
    v = inputs.views(rng, P, D, pixel)
    bank = gpu_lib.pose_bank(**mixture_args(g), rot=dev(inputs.haar_rotations(rng, K).astype(np.float32)),
                             n_psi=0, D=D, pixel=pixel)
    Y = dev(rng.standard_normal((P, D, D)).astype(np.float32))

    def search(n):
        batch = gpu_lib.pose_batch(D, pixel, n, r)
        batch.load(Y[:n].contiguous(), ctf_arg(v.subset(np.arange(n))))
        out = batch.search(bank, want_scores=True)
        torch.cuda.synchronize()
        got = out["scores"].clone(), out["rot_idx"].clone(), out["shift_idx"].clone()
        batch.close()
        return got

    announce(f"search of {P} particles, D={D}, K={K}")
    whole = search(P)
    for n in sizes:
        announce(f"  of {n}")
        small = search(n)
        for a, b in zip(small, whole):
            assert torch.equal(a, b[:n])
    bank.close()
