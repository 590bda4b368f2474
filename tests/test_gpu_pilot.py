"""Pilots counted four queries to a block (batches above 256 queries) against each query's own: the quantizer's outputs, the
bound among them, are defined bit for bit, so both give the same bytes.  Lengths around the least pilot and the rounds of a
block, batches that leave a block's last places empty, crowds of equal codes (fewer different keys than results)."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

LAYOUTS = {"16x4": ([4] * 16, 8), "16x4w": ([4] * 16, 16), "32x4": ([4] * 32, 8), "32x4w": ([4] * 32, 16), "664": ([6, 6, 4] * 4, 16),
           "664n": ([6, 6, 4] * 4, 8), "40": ([6, 5, 5, 6, 5, 5, 4, 4], 16), "35": ([5] * 7, 8), "664x2": ([6, 6, 4] * 8, 16),
           "8x8": ([8] * 8, 16), "16x8": ([8] * 16, 16)}


@pytest.mark.parametrize("crowd", [False, True])
@pytest.mark.parametrize("name", list(LAYOUTS))
def test_shared_pilot_gives_each_querys_bound(name, crowd):
    from paper_1812_09162_amd import binding as qb
    nbits, acc = LAYOUTS[name]
    d, B = 64, sum(nbits)
    rng = np.random.default_rng(B + acc + crowd)
    dsub = [d * b // B for b in nbits]
    dsub[0] += d - sum(dsub)
    dev = torch.device("cuda:0")
    cb = torch.from_numpy(rng.standard_normal(sum((1 << b) * s for b, s in zip(nbits, dsub))).astype(np.float32)).to(dev)
    idx = qb.PqIndex(d, nbits, dsub, cb, acc)
    queries = torch.from_numpy(rng.standard_normal((261, d)).astype(np.float32)).to(dev)
    tables = qb.pq_compute_tables(idx, queries)
    for n in (16383, 16384, 16385, 20480, 65535, 66001):
        codes = rng.integers(0, 256, (5 if crowd else n, (B + 7) // 8), dtype=np.uint8)
        if B % 8:
            codes[:, -1] &= (1 << (B % 8)) - 1
        codes = torch.from_numpy(codes[np.arange(n) % codes.shape[0]]).to(dev)
        for R in (1, 100, 700):
            many = qb.pq_quantize_tables(idx, tables, codes, 400, R)
            own = [qb.pq_quantize_tables(idx, tables[a:b].contiguous(), codes, 400, R) for a, b in ((0, 100), (100, 261))]
            for i in range(2):
                want = torch.cat([o[i].contiguous().view(torch.uint8) for o in own])
                assert torch.equal(many[i].contiguous().view(torch.uint8), want), (n, R, i)
    idx.close()
