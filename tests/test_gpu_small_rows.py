"""Rows far below a codebook's largest gain, at several scales of the codebook:
every path that decides rows by the float16 contraction keeps the interface's
margin (indices agree wherever the top two scores differ by more than 1e-4 of
the row's energy; below that the choice is within it).

One codeword has a gain near 2^ex, the others and the rows lie around 2^(ex +
lg).  Float16 rows go down to subnormal elements.
"""
import numpy as np
import pytest
import torch

from oracle import gsrq_oracle as O
from paper_2607_01065_amd import gsrq as B
from tests.gpu_util import check_assignment

pytestmark = pytest.mark.gpu

# (ex, lg): largest gains of about 2^5, 1, 2^-6, 2^-10 and 2^-13
SCALES16 = [(5, -8), (5, -14), (5, -18), (0, -8), (0, -12), (0, -14), (0, -20), (-6, -8), (-6, -10), (-6, -13),
            (-10, -4), (-10, -8), (-13, -6)]
SCALES32 = [(5, -10), (0, -13), (0, -17), (0, -20), (-6, -18), (-10, -20)]


def _case(N, G, d, K, ex, lg, dtype):
    rng = np.random.default_rng([N, d, K, ex + 50, lg + 50])
    shape = rng.standard_normal((G, K, d))
    shape /= np.linalg.norm(shape, axis=-1, keepdims=True)
    gain = 2.0 ** (ex + lg) * rng.uniform(0.5, 2.0, (G, K))
    gain[:, 0] = 0.9 * 2.0 ** ex
    gain, shape = gain.astype(np.float32), shape.astype(np.float32)
    X = np.empty((N, G, d))
    for g in range(G):
        k = rng.integers(1, K, N)
        X[:, g] = gain[g, k, None] * shape[g, k] * rng.uniform(0.6, 1.4, (N, 1))
    X += 2.0 ** (ex + lg - 1) * rng.standard_normal((N, G, d)) / np.sqrt(d)
    X[-1] = 0.0
    return X.reshape(N, G * d).astype(dtype), gain, shape


def _check(X, gain, shape, k, what):
    G, K, d = shape.shape
    for g in range(G):
        check_assignment(X[:, g * d:(g + 1) * d], gain[g].astype(np.float64), shape[g].astype(np.float64), k[:, g], what)


@pytest.mark.parametrize("dtype,scales", [(np.float16, SCALES16), (np.float32, SCALES32)])
@pytest.mark.parametrize("d,K,N", [
    (8, 256, 600), (4, 32, 600),             # narrow family
    (8, 512, 700), (16, 256, 600),           # resident tables
    (32, 256, 500),                          # streamed tables
    (64, 256, 600), (128, 256, 600),         # whole table in LDS, stage-fused encode
    (256, 256, 300),                         # streamed, one row block a round
    (64, 1024, 1100), (128, 1024, 1100),     # single pass and listed rows
])
def test_small_rows_keep_the_margin(d, K, N, dtype, scales):
    G = 2
    for ex, lg in scales:
        X, gain, shape = _case(N, G, d, K, ex, lg, dtype)
        what = f"d {d} K {K} {np.dtype(dtype).name} gain 2^{ex} rows 2^{ex + lg}"
        Xd, gd, sd = (torch.from_numpy(a).cuda() for a in (X, gain, shape))
        codes, _ = B.encode(Xd, gd[None], sd[None])
        X64 = X.astype(np.float64)
        k = O.unpack_codes(codes.cpu().numpy().view(np.uint32), 1, G, K)[:, 0]
        _check(X64, gain, shape, k, "encode " + what)
        r = B.train_stage(Xd, d, K, 1, gain=gd.clone(), shape=sd.clone(), resume=True, no_early_stop=True)
        _check(X64, gain, shape, r.assign.cpu().numpy().view(np.uint16).astype(np.int64).T, "train " + what)
        if d <= 8 and K <= 256:
            codes, _ = B.encode_prepared(Xd[:100], B.prepare_codebook(gd[None], sd[None]))
            k = O.unpack_codes(codes.cpu().numpy().view(np.uint32), 1, G, K)[:, 0]
            _check(X64[:100], gain, shape, k, "append " + what)
