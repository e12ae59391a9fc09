"""Decode with the codebook slices in LDS (d >= 64, several stages, many rows):
the same values, bit for bit, as the gather kernel gives for row ranges too
small for it, and the decode contract (float32 codewords, summed in stage
order in float32) in numpy."""
import numpy as np
import pytest
import torch

from paper_2607_01065_amd import gsrq as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,D,d,K,M,M_use,dtype,pad", [
    (4096, 1024, 128, 256, 12, 12, torch.float16, 0), (4097, 1024, 64, 256, 4, 4, torch.float32, 0),
    (12345, 512, 128, 128, 17, 17, torch.float16, 8), (9001, 768, 256, 256, 33, 32, torch.float32, 4),
    (33000, 128, 128, 256, 5, 4, torch.float16, 0), (20011, 1024, 256, 128, 6, 6, torch.float16, 0),
])
def test_decode_table_matches_gather_and_contract(N, D, d, K, M, M_use, dtype, pad):
    G, b = D // d, int(np.log2(K))
    rng = np.random.default_rng(N + M)
    gain = torch.from_numpy(rng.lognormal(0, 0.5, (M, G, K)).astype(np.float32)).cuda()
    shape = torch.from_numpy(rng.standard_normal((M, G, K, d)).astype(np.float32)).cuda()
    words = torch.from_numpy(rng.integers(0, 2 ** 32, (N, (M * G * b + 31) // 32), dtype=np.uint32)
                             .view(np.int32)).cuda()
    full = torch.full((N, D + pad), 7.0, dtype=dtype, device="cuda")
    out = B.decode(words, gain, shape, D, M_use, out=full[:, :D])
    assert pad == 0 or bool((full[:, D:] == 7.0).all())
    step = 1000                               # few rows: the gather kernel
    for r in range(0, N, step):
        assert torch.equal(B.decode(words[r:r + step].contiguous(), gain, shape, D, M_use, out_dtype=dtype),
                           out[r:r + step])
    rows = np.unique(np.concatenate([[0, N - 1], rng.integers(0, N, 40)]))
    bits = np.unpackbits(words[torch.from_numpy(rows).cuda()].cpu().numpy().view(np.uint8), axis=1,
                         bitorder="little")[:, : M * G * b].reshape(len(rows), M, G, b)
    k = (bits.astype(np.int64) << np.arange(b)).sum(-1)
    book = gain.cpu().numpy()[..., None] * shape.cpu().numpy()
    want = np.zeros((len(rows), G, d), np.float32)
    for m in range(M_use):
        want += book[m, np.arange(G), k[:, m]]
    got = out[torch.from_numpy(rows).cuda()].cpu().numpy()
    assert np.array_equal(got, want.reshape(len(rows), D).astype(got.dtype))
