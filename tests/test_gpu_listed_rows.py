"""Rows that the large-codebook single pass lists (K >= 1024): outputs written by
the finish kernel, on aligned and unaligned rows.

Gaussian rows against random codewords leave many rows within the single
pass's error bound, so a large share of them takes the listed path.
"""
import numpy as np
import pytest
import torch

import synth
from oracle import gsrq_oracle as O
from paper_2607_01065_amd import gsrq as B

pytestmark = pytest.mark.gpu


def _rows(X, pad, dtype):
    """X on the device with `pad` unused elements at the end of every row."""
    full = torch.zeros((X.shape[0], X.shape[1] + pad), dtype=dtype, device="cuda")
    full[:, : X.shape[1]] = torch.from_numpy(X).cuda().to(dtype)
    return full[:, : X.shape[1]]


@pytest.mark.parametrize("d,K,pad,dtype", [
    (64, 1024, 0, torch.float32), (128, 1024, 0, torch.float16), (128, 2048, 3, torch.float32),
    (256, 1024, 0, torch.float32), (64, 1024, 1, torch.float16),
])
def test_listed_rows_objective_codes_residual(d, K, pad, dtype):
    N, G = 4 * K + 37, 2
    X, w, seeds = synth.small_case(N, G * d, d, K, 1, seed=d + K, key_sigma=0.0)
    if dtype == torch.float16:
        X = X.astype(np.float16).astype(np.float32)
    Xd = _rows(X, pad, dtype)
    wd = torch.from_numpy(w).cuda()
    init = B.train_stage(Xd, d, K, 0, seed_rows=seeds[0], w=wd)
    gain, shape = init.gain.clone(), init.shape.clone()
    r = B.train_stage(Xd, d, K, 1, w=wd, gain=init.gain, shape=init.shape, resume=True,
                      no_early_stop=True)
    codes, res = B.encode(Xd, gain[None], shape[None], residual=True)
    torch.cuda.synchronize()
    g64, s64 = gain.cpu().numpy().astype(np.float64), shape.cpu().numpy().astype(np.float64)
    assign = r.assign.cpu().numpy().view(np.uint16).astype(np.int64)
    k_enc = O.unpack_codes(codes.cpu().numpy().view(np.uint32), 1, G, K)[:, 0]
    X64 = X.astype(np.float64)
    for g in range(G):
        Xg = X64[:, g * d:(g + 1) * d]
        best = np.argmax(O.gskm_scores(Xg, g64[g], s64[g]), axis=1)
        clear = O.assignment_margin(Xg, g64[g], s64[g]) > 1e-4
        assert np.array_equal(assign[g][clear], best[clear])
        assert np.array_equal(k_enc[clear, g], best[clear])
        # float64 sums of the rows' energies
        diff = Xg - g64[g][assign[g], None] * s64[g][assign[g]]
        want = float(np.sum(w.astype(np.float64) * np.sum(diff * diff, axis=1)))
        energy = float(np.sum(w.astype(np.float64) * np.sum(Xg * Xg, axis=1)))
        assert abs(float(r.trace[g, 0]) - want) <= N * 2.0 ** -52 * energy
        # one float32 multiply-add per element
        ref = Xg - g64[g][k_enc[:, g], None] * s64[g][k_enc[:, g]]
        got = res[:, g * d:(g + 1) * d].cpu().numpy()
        assert np.max(np.abs(got - ref)) <= 2.0 ** -23 * np.max(np.abs(Xg) + np.abs(ref))


@pytest.mark.parametrize("d,K,dtype", [
    (64, 1024, torch.float16), (128, 1024, torch.float32), (128, 2048, torch.float16), (256, 1024, torch.float32),
])
def test_single_pass_bounds_over_wide_scales(d, K, dtype):
    """Gains over two decades, rows from well below to far above them, rows
    on top of codewords, duplicated codewords and zero rows: no row is decided
    wrongly above the margin, and exact ties go to the lowest index."""
    N, G = 4096, 2
    rng = np.random.default_rng(d + K)
    shape = rng.standard_normal((1, G, K, d))
    shape = (shape / np.linalg.norm(shape, axis=-1, keepdims=True)).astype(np.float32)
    gain = rng.lognormal(0.0, 1.0, (1, G, K)).astype(np.float32)
    gain[0, :, K // 2:K // 2 + 8] = gain[0, :, :8]           # codewords 0..7 again at K / 2
    shape[0, :, K // 2:K // 2 + 8] = shape[0, :, :8]
    X = rng.standard_normal((N, G, d)) * 2.0 ** rng.uniform(-6, 6, (N, G, 1)) / np.sqrt(d)
    X[:K // 2] = (gain[0, :, :K // 2, None] * shape[0, :, :K // 2]).transpose(1, 0, 2)
    X[-16:] = 0.0
    Xd = torch.from_numpy(X.reshape(N, G * d)).to(dtype).cuda()
    codes, _ = B.encode(Xd, torch.from_numpy(gain).cuda(), torch.from_numpy(shape).cuda())
    k = O.unpack_codes(codes.cpu().numpy().view(np.uint32), 1, G, K)[:, 0]
    X64 = Xd.double().cpu().numpy()
    for g in range(G):
        Xg = X64[:, g * d:(g + 1) * d]
        S = O.gskm_scores(Xg, gain[0, g], shape[0, g])
        clear = O.assignment_margin(Xg, gain[0, g], shape[0, g]) > 1e-4
        assert np.array_equal(k[clear, g], np.argmax(S, axis=1)[clear])
        assert np.all(k[:8, g] == np.arange(8))              # equal codewords: the lower index
