"""One-launch bucketing of the sorted sums: a training iteration at row counts
and codebook sizes at its edges gives the codewords that the members' float64
sums give (every row in its codeword's bucket exactly once)."""
import numpy as np
import pytest
import torch

from oracle import gsrq_oracle as O
from paper_2607_01065_amd import gsrq as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,d,K,skew", [
    (16384, 128, 256, False), (16385, 128, 256, True), (2049, 64, 512, True), (8191, 128, 512, False),
    (65536, 64, 2048, True), (65529, 64, 4096, False), (65537, 64, 2048, False), (4100, 256, 64, True),
])
def test_update_from_bucketed_rows(N, d, K, skew):
    G = 2
    rng = np.random.default_rng(N + K)
    # rows near a codeword each, so that the assignment is known; skew: half of them on codeword 3
    shape = rng.standard_normal((G, K, d))
    shape /= np.linalg.norm(shape, axis=-1, keepdims=True)
    k = rng.integers(0, K, (G, N))
    if skew:
        k[:, rng.permutation(N)[: N // 2]] = 3
    X = np.concatenate([shape[g, k[g]] for g in range(G)], axis=1) + 1e-3 * rng.standard_normal((N, G * d))
    X = X.astype(np.float32)
    w = rng.lognormal(0.0, 1.0, N).astype(np.float32)
    st = torch.from_numpy(shape.astype(np.float32)).cuda()
    r = B.train_stage(torch.from_numpy(X).cuda(), d, K, 1, w=torch.from_numpy(w).cuda(),
                      gain=torch.ones((G, K), device="cuda"), shape=st.clone(), resume=True,
                      no_early_stop=True)
    s32 = st.double().cpu().numpy()
    for g in range(G):
        assign = r.assign[g].cpu().numpy().view(np.uint16).astype(np.int64)
        assert np.array_equal(assign, k[g])
        gain, sh = O.gskm_update(X[:, g * d:(g + 1) * d], w, assign, np.ones(K), s32[g])
        # float32 products w y and a float32 result; a row more or less in a bucket shows at 1e-4
        assert np.max(np.abs(r.gain[g].cpu().numpy() - gain)) <= 4 * 2.0 ** -24
        assert np.max(np.abs(r.shape[g].cpu().numpy() - sh)) <= 8 * 2.0 ** -24
