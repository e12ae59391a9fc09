"""Training pass with the whole codebook table in LDS (d = 64 and 128): row
counts at the edges of 32-row blocks and of the workgroups' shares, and the
same rows at an alignment that takes the streamed kernel instead."""
import numpy as np
import pytest
import torch

import synth
from oracle import gsrq_oracle as O
from paper_2607_01065_amd import gsrq as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,G,d,K,dtype", [
    (256, 1, 128, 128, torch.float32), (257, 3, 128, 256, torch.float32), (2049, 2, 128, 256, torch.float16),
    (8191, 8, 128, 256, torch.float32), (1025, 2, 64, 256, torch.float16), (1023, 3, 64, 512, torch.float32),
])
def test_table_pass_against_streamed_and_oracle(N, G, d, K, dtype):
    X, w, seeds = synth.small_case(N, G * d, d, min(K, N), 1, seed=N + d, key_sigma=0.5)
    gain = np.linalg.norm(X.reshape(N, G, d)[seeds[0].T % N, np.arange(G)], axis=-1).T[:, :K]
    Xt = torch.from_numpy(X).cuda().to(dtype)
    X64 = Xt.double().cpu().numpy()
    rng = np.random.default_rng(N)
    shape = rng.standard_normal((G, K, d))
    shape /= np.linalg.norm(shape, axis=-1, keepdims=True)
    gain = np.resize(gain, (G, K)) * rng.uniform(0.2, 1.0, (G, K))
    gt = torch.from_numpy(gain.astype(np.float32)).cuda()
    st = torch.from_numpy(shape.astype(np.float32)).cuda()
    padded = torch.zeros((N, G * d + 1), dtype=dtype, device="cuda")   # rows off 16-byte alignment
    padded[:, : G * d] = Xt
    out = []
    for rows in (Xt, padded[:, : G * d]):
        r = B.train_stage(rows, d, K, 1, w=torch.from_numpy(w).cuda(), gain=gt.clone(), shape=st.clone(),
                          resume=True, no_early_stop=True)
        out.append(r.assign.cpu().numpy().view(np.uint16).astype(np.int64))
    assert np.array_equal(out[0], out[1])        # the same operands, products and keys
    g64, s64 = gt.double().cpu().numpy(), st.double().cpu().numpy()
    for g in range(G):
        Xg = X64[:, g * d:(g + 1) * d]
        clear = O.assignment_margin(Xg, g64[g], s64[g]) > 1e-4
        best = np.argmax(O.gskm_scores(Xg, g64[g], s64[g]), axis=1)
        assert np.array_equal(out[0][g][clear], best[clear])


def test_table_pass_stop_test():
    """A repeated assignment stops the subspace; one changed row does not."""
    N, d, K = 4096, 128, 256
    X, w, seeds = synth.small_case(N, 2 * d, d, K, 1, seed=3)
    Xt, wt = torch.from_numpy(X).cuda(), torch.from_numpy(w).cuda()
    r = B.train_stage(Xt, d, K, 60, seed_rows=seeds[0], w=wt)
    it = int(r.iters.max())
    assert it < 60
    again = B.train_stage(Xt, d, K, 5, w=wt, gain=r.gain.clone(), shape=r.shape.clone(),
                          assign=r.assign.clone(), resume=True, assign_in=True)
    assert int(again.iters.max()) == 1
    moved = r.assign.clone()
    moved[1, N - 1] = (moved[1, N - 1] + 1) % K
    again = B.train_stage(Xt, d, K, 5, w=wt, gain=r.gain.clone(), shape=r.shape.clone(),
                          assign=moved, resume=True, assign_in=True)
    assert again.iters.tolist() == [1, 2]
