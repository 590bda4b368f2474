"""Lists longer than a pair's slot list is deep: the scan cuts the slots back to the codes up to the R-th distance (or, with
crowds of equal distances, leaves the selection to a pass over the codes).  Compared with the oracle, bit for bit: layouts of
every scan kind, lists around the slots' depth and its multiples, results on both sides of the depths and block sizes."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu

LAYOUTS = {"16x4": ([4] * 16, 8, 96), "32x4": ([4] * 32, 8, 64), "664": ([6, 6, 4] * 4, 16, 48), "40": ([6, 5, 5, 6, 5, 5, 4, 4], 16, 48),
           "8x8": ([8] * 8, 16, 32), "odd": ([3, 5, 7, 2], 8, 20)}


@pytest.mark.parametrize("kind", ["random", "few different", "equal"])
@pytest.mark.parametrize("R", [1, 100, 128, 129, 700])
@pytest.mark.parametrize("name", list(LAYOUTS))
def test_long_lists(name, R, kind):
    from paper_1812_09162_amd import binding as qb
    nbits, acc, d = LAYOUTS[name]
    rng = np.random.default_rng(R + len(name))
    B = sum(nbits)
    dsub = [d * b // B for b in nbits]
    dsub[0] += d - sum(dsub)
    lens = [1023, 1024, 1025, 0, 60_001, 3, 4097, 30_000]
    n, K = sum(lens), len(lens)
    cb = rng.standard_normal(sum((1 << b) * s for b, s in zip(nbits, dsub))).astype(np.float32)
    coarse = (0.3 * rng.standard_normal((K, d))).astype(np.float32)
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    codes = rng.integers(0, 256, (n, (B + 7) // 8), dtype=np.uint8)
    if B % 8:
        codes[:, -1] &= (1 << (B % 8)) - 1
    if kind != "random":
        codes = codes[rng.integers(0, 9, n) if kind == "few different" else np.zeros(n, dtype=np.int64)]
    ids = rng.permutation(n).astype(np.int32)
    q = rng.standard_normal((3, d)).astype(np.float32)
    probe = np.stack([rng.permutation(K) for _ in range(3)]).astype(np.int32)
    dev = torch.device("cuda:0")
    idx = qb.PqIndex(d, nbits, dsub, torch.from_numpy(cb).to(dev), acc)
    args = [idx] + [torch.from_numpy(np.ascontiguousarray(x)).to(dev) for x in (coarse, off, codes, ids, q, probe)] + [400, R]
    gi, gd = qb.ivf_adc_scan_topk(*args)
    qb.pq_set_option(qb.PQ_OPT_IVF_SHARED_LISTS, 2)
    try:
        si, sd = qb.ivf_adc_scan_topk(*args)
    finally:
        qb.pq_set_option(qb.PQ_OPT_IVF_SHARED_LISTS, 1)
    torch.cuda.synchronize()
    assert torch.equal(gi, si) and torch.equal(gd, sd)
    for a in range(3):
        oi, od, _ = oracle.search_ivf(d, nbits, dsub, acc, cb, coarse, off, codes, ids, q[a], probe[a], 400, R)
        assert np.array_equal(gi[a].cpu().numpy(), oi) and np.array_equal(gd[a].cpu().numpy(), od), a
    idx.close()
