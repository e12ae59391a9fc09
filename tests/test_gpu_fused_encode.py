"""Stage-fused encode at d = 64 and 128 (hi/lo contraction over a stage's table in
LDS): equal and nearly equal codewords, zero gains, single tiles and the
largest tables, odd row counts, against the float64 residual recursion stage by
stage."""
import numpy as np
import pytest
import torch

from oracle import gsrq_oracle as O
from paper_2607_01065_amd import gsrq as B

pytestmark = pytest.mark.gpu


def _check(X, gain, shape, codes):
    """Every stage's code, given the codes before it: the argmax above the
    margin, within the margin of it below."""
    M, G, K = gain.shape
    d = shape.shape[-1]
    k = O.unpack_codes(codes.cpu().numpy().view(np.uint32), M, G, K)
    for g in range(G):
        r = X[:, g * d:(g + 1) * d].astype(np.float64)
        for m in range(M):
            S = O.gskm_scores(r, gain[m, g], shape[m, g])
            got = np.take_along_axis(S, k[:, m, g:g + 1], 1)[:, 0]
            energy = np.maximum(np.sum(r * r, axis=1), 1e-30)
            assert np.all(S.max(axis=1) - got <= 1e-4 * energy), (m, g)
            # the float32 residual that the kernel carries
            r = (r - gain[m, g, k[:, m, g], None].astype(np.float64) * shape[m, g, k[:, m, g]])
            r = r.astype(np.float32).astype(np.float64)
    return k


@pytest.mark.parametrize("d,K,M,N,dtype,pad", [
    # a workgroup (256 rows of a subspace) for every CU: one row in the last, full ones, a partial block; unaligned rows
    (128, 256, 3, 127 * 256 + 1, torch.float16, 0), (128, 256, 2, 32768, torch.float32, 3),
    (64, 512, 3, 128 * 256 - 31, torch.float16, 0),
    # a few workgroups, single tiles (K = 32), less than a block
    (128, 256, 3, 257, torch.float16, 0), (128, 32, 2, 100, torch.float32, 0), (64, 512, 3, 300, torch.float16, 0),
    (64, 256, 5, 33, torch.float32, 0), (64, 32, 2, 31, torch.float16, 1),
])
def test_fused_encode_open_rows(d, K, M, N, dtype, pad):
    G = 2
    rng = np.random.default_rng(d + K + N)
    shape = rng.standard_normal((M, G, K, d))
    shape /= np.linalg.norm(shape, axis=-1, keepdims=True)
    gain = 0.5 ** np.arange(M)[:, None, None] * rng.uniform(0.3, 1.0, (M, G, K))
    q = K // 4
    gain[:, :, q:2 * q] = gain[:, :, :q]                     # pairs that agree to 1e-3, 1e-6 and exactly
    eps = np.resize([1e-3, 1e-6, 0.0], q)[:, None]
    shape[:, :, q:2 * q] = shape[:, :, :q] + eps * rng.standard_normal((M, G, q, d)) / np.sqrt(d)
    gain[:, :, 2 * q:2 * q + 5] = gain[:, :, :1]             # more than three nearly equal
    shape[:, :, 2 * q:2 * q + 5] = shape[:, :, :1] + 1e-5 * rng.standard_normal((M, G, 5, d)) / np.sqrt(d)
    same = np.flatnonzero(eps[:, 0] == 0.0)
    exact = shape[:, :, same]
    shape /= np.linalg.norm(shape, axis=-1, keepdims=True)   # unit rows, as codebooks hold them
    shape[:, :, same] = shape[:, :, same + q] = exact
    gain[:, :, 3 * q:3 * q + 6] = 0.0                        # several zero gains
    gain, shape = gain.astype(np.float32), shape.astype(np.float32)
    rows = rng.integers(0, K, (N, G))
    X = np.concatenate([gain[0, g, rows[:, g], None] * shape[0, g, rows[:, g]] for g in range(G)], axis=1)
    X = X + 0.05 * rng.standard_normal((N, G * d)) * rng.integers(0, 2, (N, 1))
    X[-3:] = 0.0
    full = torch.zeros((N, G * d + pad), dtype=dtype, device="cuda")
    full[:, : G * d] = torch.from_numpy(X).cuda().to(dtype)
    Xd = full[:, : G * d]
    codes, res = B.encode(Xd, torch.from_numpy(gain).cuda(), torch.from_numpy(shape).cuda(), residual=True)
    X64 = Xd.double().cpu().numpy()
    k = _check(X64, gain, shape, codes)
    # a row on an exactly repeated codeword goes to the lower index
    for g in range(G):
        assert not np.any(np.isin(k[:, 0, g], same + q))
        assert not np.any(np.isin(k[:, :, g], np.arange(3 * q + 1, 3 * q + 6)))   # the first zero gain only
    want = X64 - O.gsrq_decode(k, gain.astype(np.float64), shape.astype(np.float64))
    scale = np.max(np.abs(X64)) + np.max(gain)
    assert np.max(np.abs(res.cpu().numpy() - want)) <= 2 * M * 2.0 ** -24 * scale
