"""Objective trace of the wide family, formed from the codewords' float64 sums:
against the distortion of the same assignment summed row by row in float64.

The rows lie close to their codewords (energy about 10^4 times the
distortion), so the difference of sums would show any rounding of its terms.
"""
import numpy as np
import pytest
import torch

from paper_2607_01065_amd import gsrq as B

pytestmark = pytest.mark.gpu


def _clusters(N, G, d, K, seed, dtype):
    rng = np.random.default_rng(seed)
    c = rng.standard_normal((K, G * d)) * rng.lognormal(0.0, 0.5, size=(K, 1))
    X = c[rng.integers(0, K, N)] + 1e-2 * rng.standard_normal((N, G * d))
    X[:K] = c          # every cluster has a member to start from
    return X.astype(dtype), rng.lognormal(0.0, 1.0, N).astype(np.float32)


@pytest.mark.parametrize("d,K,N,dtype,kmeans", [
    (16, 32, 1000, np.float32, False), (16, 256, 5000, np.float16, False), (8, 512, 4099, np.float32, False),
    (32, 64, 3001, np.float32, True), (64, 256, 2000, np.float32, False), (128, 256, 4001, np.float16, True),
    (128, 1024, 5003, np.float32, False), (256, 64, 1500, np.float32, False), (256, 64, 1500, np.float32, True),
])
def test_trace_is_the_distortion(d, K, N, dtype, kmeans):
    G, T = 2, 3
    X, w = _clusters(N, G, d, K, 7 * d + K, dtype)
    seeds = np.stack([np.random.default_rng(g).permutation(K) for g in range(G)])
    Xd, wd = torch.from_numpy(X).cuda(), torch.from_numpy(w).cuda()
    kw = dict(seed_rows=seeds, w=wd, no_early_stop=True, kmeans=kmeans)
    full = B.train_stage(Xd, d, K, T, **kw)
    before = B.train_stage(Xd, d, K, T - 1, **kw)
    book = full if kmeans else before      # the codebook the last entry is measured against
    torch.cuda.synchronize()
    w64 = w.astype(np.float64)
    for g in range(G):
        Xg = X[:, g * d:(g + 1) * d].astype(np.float64)
        k = full.assign[g].cpu().numpy().view(np.uint16).astype(np.int64)
        c = (book.gain[g][:, None].double() * book.shape[g].double()).cpu().numpy()
        want = float(np.sum(w64 * np.sum((Xg - c[k]) ** 2, axis=1)))
        energy = float(np.sum(w64 * np.sum(Xg * Xg, axis=1)))
        # float64 sums of at most N d terms of one sign; K-means: the float32
        # rounding of the centroids enters squared
        bound = N * 2.0 ** -52 * energy + (2.0 ** -44 * energy if kmeans else 0.0)
        assert abs(float(full.trace[g, T - 1]) - want) <= bound
        assert full.iters[g] == T


@pytest.mark.parametrize("d,K", [(16, 32), (128, 64)])
def test_trace_ends_where_the_subspace_stops(d, K):
    X, w = _clusters(2000, 3, d, K, 5, np.float32)
    seeds = np.tile(np.arange(K), (3, 1))
    r = B.train_stage(torch.from_numpy(X).cuda(), d, K, 12, seed_rows=seeds,
                      w=torch.from_numpy(w).cuda())
    torch.cuda.synchronize()
    it, tr = r.iters.cpu().numpy(), r.trace.cpu().numpy()
    assert np.all(it < 12)
    for g in range(3):
        assert np.all(tr[g, :it[g]] > 0) and np.all(tr[g, it[g]:] == 0)


@pytest.mark.parametrize("kmeans", [False, True])
@pytest.mark.parametrize("near", [0.0, 2.0 ** -9, 2.0 ** -7])
@pytest.mark.parametrize("d,K,N,pad,dtype", [
    (16, 256, 3000, 0, np.float32), (16, 64, 1000, 0, np.float16), (8, 512, 2000, 0, np.float32),  # sums in LDS
    (64, 256, 2000, 0, np.float32), (128, 256, 3000, 0, np.float32), (128, 256, 2000, 0, np.float16),  # sorted sums
    (128, 8, 2000, 0, np.float32),           # crowded codewords: windows of the sorted sums
    (128, 256, 2000, 3, np.float32),         # unaligned rows: sliced sums in LDS
    (256, 256, 1000, 0, np.float32), (256, 256, 1000, 1, np.float32), (128, 1024, 3000, 0, np.float32),
])
def test_trace_of_rows_on_their_codewords(d, K, N, pad, dtype, near, kmeans):
    """The codebook reproduces half of its members to their rounding (distortion
    about 1e-15 of the energy, 1e-7 in float16) and half to a relative `near`:
    the trace is right relative to itself."""
    G = 2
    rng = np.random.default_rng([d, K, N, pad])
    gain = rng.lognormal(0.0, 0.3, (G, K)).astype(np.float32)
    shape = rng.standard_normal((G, K, d))
    shape = (shape / np.linalg.norm(shape, axis=-1, keepdims=True)).astype(np.float32)
    c = gain[..., None].astype(np.float64) * shape
    k = rng.integers(0, K, (N, G))
    X = np.stack([c[g, k[:, g]] for g in range(G)], axis=1)
    X += near * (k >= K // 2)[..., None] * rng.standard_normal((N, G, d)) / np.sqrt(d)
    X = X.reshape(N, G * d).astype(dtype)
    w = rng.lognormal(0.0, 1.0, N).astype(np.float32)
    full = torch.zeros((N, G * d + pad), dtype=torch.from_numpy(X).dtype, device="cuda")
    full[:, : G * d] = torch.from_numpy(X)
    r = B.train_stage(full[:, : G * d], d, K, 1, w=torch.from_numpy(w).cuda(), resume=True, no_early_stop=True,
                      kmeans=kmeans, gain=torch.from_numpy(gain).cuda(), shape=torch.from_numpy(shape).cuda())
    X64, w64 = X.astype(np.float64).reshape(N, G, d), w.astype(np.float64)[:, None]
    for g in range(G):
        assert np.array_equal(r.assign[g].cpu().numpy().view(np.uint16), k[:, g])
        before = float(np.sum(w64 * (X64[:, g] - c[g, k[:, g]]) ** 2))
        if kmeans:
            mass = np.maximum(np.bincount(k[:, g], w64[:, 0], K), 1e-30)[:, None]
            # from the codeword, so that the mean keeps its digits
            off = np.zeros((K, d))
            np.add.at(off, k[:, g], w64 * (X64[:, g] - c[g, k[:, g]]))
            want = float(np.sum(w64 * (X64[:, g] - c[g, k[:, g]] - (off / mass)[k[:, g]]) ** 2))
        else:
            want = before
        # float64 sums: N d terms of one sign, or 2^16 times that where they are a difference of energies; the means
        # of K-means are rounded to 2^-53 of the rows, whose squares enter
        energy = float(np.sum(w64 * X64[:, g] ** 2))
        bound = N * 2.0 ** -52 * (d * before + min(energy, 2.0 ** 16 * before) * (near > 0.0))
        bound += 2.0 ** -50 * np.sqrt(before * energy) if kmeans else 0.0
        got = float(r.trace[g, 0])
        assert 0.0 <= got and abs(got - want) <= bound, (got, want)
