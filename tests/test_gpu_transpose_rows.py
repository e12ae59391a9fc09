"""Subspace-major copy of the narrow training call (d = 8): whole 16-byte rows and
rows off that alignment give the same assignment and codebook, at row and
subspace counts that leave partial groups of eight."""
import numpy as np
import pytest
import torch

import synth
from paper_2607_01065_amd import gsrq as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,G,dtype", [
    (257, 3, torch.float16), (2049, 16, torch.float32), (33001, 130, torch.float16), (16385, 72, torch.float32),
])
def test_aligned_and_unaligned_rows_agree(N, G, dtype):
    K = 64
    X, w, seeds = synth.small_case(N, G * 8, 8, K, 1, seed=N)
    Xt = torch.from_numpy(X).cuda().to(dtype)
    padded = torch.zeros((N, G * 8 + 1), dtype=dtype, device="cuda")
    padded[:, : G * 8] = Xt
    wt = torch.from_numpy(w).cuda()
    a, b = (B.train_stage(rows, 8, K, 2, seed_rows=seeds[0], w=wt, no_early_stop=True)
            for rows in (Xt, padded[:, : G * 8]))
    assert np.array_equal(a.assign.cpu().numpy(), b.assign.cpu().numpy())
    # the same rows; float64 sums in another order before float32 rounding
    assert torch.allclose(a.gain, b.gain, rtol=2.0 ** -22, atol=0)
    assert torch.allclose(a.shape, b.shape, rtol=0, atol=2.0 ** -22)
