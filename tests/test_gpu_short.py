"""Searches whose list the quantizer's blocks scan themselves (k_quantize_short), against the same search stage by stage: both
are defined bit for bit.  Lengths around the slices and the longest such list, results around the longest list of a block,
crowds of equal keys (fewer whole bins than results), and a list whose nearest codes all lie in one slice."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu

LAYOUTS = {"16x4": ([4] * 16, 8), "16x4w": ([4] * 16, 16), "32x4": ([4] * 32, 8), "664": ([6, 6, 4] * 4, 16), "40": ([6, 5, 5, 6, 5, 5, 4, 4], 16),
           "664x2": ([6, 6, 4] * 8, 16), "8x8": ([8] * 8, 16), "odd": ([3, 5, 7, 2], 8)}


@pytest.mark.parametrize("kind", ["random", "few different", "equal", "one slice"])
@pytest.mark.parametrize("name", list(LAYOUTS))
def test_short_lists_match_the_stages(name, kind):
    from paper_1812_09162_amd import binding as qb
    nbits, acc = LAYOUTS[name]
    d, B = 48, sum(nbits)
    cs = (B + 7) // 8
    rng = np.random.default_rng(len(name) + acc + len(kind))
    dsub = [d * b // B for b in nbits]
    dsub[0] += d - sum(dsub)
    dev = torch.device("cuda:0")
    cb = rng.standard_normal(sum((1 << b) * s for b, s in zip(nbits, dsub))).astype(np.float32)
    idx = qb.PqIndex(d, nbits, dsub, torch.from_numpy(cb).to(dev), acc)
    q = rng.standard_normal((20, d)).astype(np.float32)
    pool = rng.integers(0, 256, (262_145, cs), dtype=np.uint8)
    if B % 8:
        pool[:, -1] &= (1 << (B % 8)) - 1
    if kind == "few different":
        pool = pool[rng.integers(0, 9, pool.shape[0])]
    if kind == "equal":
        pool[:] = pool[0]
    sizes = (1, 2, 63, 1023, 1024, 1025, 4097, 65_537, 131_071, 262_144, 262_145) if kind == "random" else (5, 3000, 70_001)
    for n in sizes:
        codes = pool[:n].copy()
        if kind == "one slice" and n > 2000:  # the first query's nearest codes side by side
            codes[1000:1300] = oracle.encode(d, nbits, dsub, cb, q[:1] + 0.01 * rng.standard_normal((300, d)).astype(np.float32))
        cd = torch.from_numpy(codes).to(dev)
        for nq, R in ((1, 100), (1, 1), (3, 153), (20, 10), (2, 154)):
            qd = torch.from_numpy(q[:nq]).to(dev)
            got = qb.pq_search_topk(idx, qd, cd, 400, R)
            tables = qb.pq_compute_tables(idx, qd)
            qt, qp = qb.pq_quantize_tables(idx, tables, cd, 400, R)
            want = qb.pq_adc_scan_topk(idx, qt, qp, cd, R)
            torch.cuda.synchronize()
            for a, b in zip(got, want):
                assert torch.equal(a.view(torch.uint8), b.view(torch.uint8)), (n, nq, R)
            if n <= 4097 and nq == 1:
                oi, ok, od = oracle.search(d, nbits, dsub, acc, cb, q[0], codes, 400, R)
                assert np.array_equal(got[0][0].cpu().numpy(), oi) and np.array_equal(got[2][0].cpu().numpy(), od)
    idx.close()
