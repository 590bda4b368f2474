"""The inverted-list calibration runs blocks of 1024, 512 or 256 threads by the number of queries: all give the same
results (defined bit for bit), for every code layout the kernel tells apart."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nbits,d,acc", [([4] * 16, 96, 8), ([4] * 16, 80, 8), ([6, 5, 5] * 4, 96, 16), ([8] * 8, 64, 16),
                                         ([4] * 40, 80, 8)])
@pytest.mark.parametrize("R", [1, 100, 600])
def test_wide_and_narrow_calibration_agree(nbits, d, acc, R):
    from paper_1812_09162_amd import binding as qb
    rng = np.random.default_rng(R + d)
    lens = [0, 1, 255, 256, 257, 1023, 1025, 90, 3000, 4500]
    K, n, nq, nprobe = len(lens), sum(lens), 513, 7
    dsub = [d // len(nbits)] * len(nbits)
    dsub[0] += d - sum(dsub)
    cb = rng.standard_normal(sum((1 << b) * s for b, s in zip(nbits, dsub))).astype(np.float32)
    coarse = rng.standard_normal((K, d)).astype(np.float32)
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    codes = rng.integers(0, 256, (n, sum(nbits) // 8), dtype=np.uint8)
    ids = rng.permutation(n).astype(np.int32)
    q = rng.standard_normal((nq, d)).astype(np.float32)
    probe = np.stack([rng.permutation(K)[:nprobe] for _ in range(nq)]).astype(np.int32)
    dev = torch.device("cuda:0")
    idx = qb.PqIndex(d, nbits, dsub, torch.from_numpy(cb).to(dev), acc)
    lists = [torch.from_numpy(x).to(dev) for x in (coarse, off, codes, ids)]
    for search in (qb.ivf_adc_scan_topk, qb.ivf_adc_scan_topk_tightening):
        many = search(idx, *lists, torch.from_numpy(q).to(dev), torch.from_numpy(probe).to(dev), 400, R)
        for k in (9, 300):
            few = search(idx, *lists, torch.from_numpy(q[:k]).to(dev), torch.from_numpy(probe[:k]).to(dev), 400, R)
            torch.cuda.synchronize()
            for a, b in zip(many, few):
                assert torch.equal(a[:k], b)
    few = qb.ivf_adc_scan_topk(idx, *lists, torch.from_numpy(q[:2]).to(dev), torch.from_numpy(probe[:2]).to(dev), 400, R)
    for i in range(2):
        oi, od, _ = oracle.search_ivf(d, nbits, dsub, acc, cb, coarse, off, codes, ids, q[i], probe[i], 400, R)
        assert np.array_equal(few[0][i].cpu().numpy(), oi) and np.array_equal(few[1][i].cpu().numpy(), od)
    idx.close()
