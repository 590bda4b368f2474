"""The quantizer's block widths: a call of a few queries runs wide blocks, one of many queries narrow ones, and both
have to give the same tables, parameters and bounds (defined bit for bit); sizes around the threads of a block."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu

LAYOUTS = {"16x4": ([4] * 16, 96, 8), "32x4": ([4] * 32, 128, 8), "664": ([6, 6, 4] * 4, 128, 16),
           "40": ([6, 5, 5, 6, 5, 5, 4, 4], 128, 16), "8x8": ([8] * 8, 128, 16), "odd": ([3, 5, 7, 2], 50, 8)}


@pytest.mark.parametrize("name", list(LAYOUTS))
@pytest.mark.parametrize("n", [1, 255, 1025, 5000])
def test_wide_and_narrow_blocks_agree(name, n):
    from paper_1812_09162_amd import binding as qb
    nbits, d, acc = LAYOUTS[name]
    rng = np.random.default_rng(n)
    B = sum(nbits)
    dsub = [d * b // B for b in nbits]
    dsub[0] += d - sum(dsub)
    cb = rng.standard_normal(sum((1 << b) * s for b, s in zip(nbits, dsub))).astype(np.float32)
    codes = rng.integers(0, 256, (n, (B + 7) // 8), dtype=np.uint8)
    if B % 8:
        codes[:, -1] &= (1 << (B % 8)) - 1
    q = rng.standard_normal((600, d)).astype(np.float32)
    dev = torch.device("cuda:0")
    idx = qb.PqIndex(d, nbits, dsub, torch.from_numpy(cb).to(dev), acc)
    cd, qd = torch.from_numpy(codes).to(dev), torch.from_numpy(q).to(dev)
    tables = qb.pq_compute_tables(idx, qd)
    for R in (1, 100, 700):
        many = qb.pq_quantize_tables(idx, tables, cd, 400, R)
        few = qb.pq_quantize_tables(idx, tables[:3].contiguous(), cd, 400, R)
        all_ = qb.pq_search_topk(idx, qd, cd, 400, R)
        one = qb.pq_search_topk(idx, qd[1:2].contiguous(), cd, 400, R)
        torch.cuda.synchronize()
        for a, b in zip(many, few):
            assert torch.equal(a[:3].contiguous().view(torch.uint8), b.contiguous().view(torch.uint8))
        for a, b in zip(all_, one):
            assert torch.equal(a[1:2], b)
        oi, ok, od = oracle.search(d, nbits, dsub, acc, cb, q[1], codes, 400, R)
        assert np.array_equal(one[0][0].cpu().numpy(), oi) and np.array_equal(one[2][0].cpu().numpy(), od)
    idx.close()
