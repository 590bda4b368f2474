"""Lists longer than a pair's slot list is deep: the scan cuts the slots back to the codes up to the R-th distance (or, with
crowds of equal distances, leaves the selection to a pass over the codes).  Compared with the oracle, bit for bit: layouts of
every scan kind, lists around the slots' depth, its multiples and the sixteen batches between two looks, results on both sides of the depths
and block sizes; lists whose near codes come last, so that every code is within the bound, and blocks of one, two and four waves."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu

LAYOUTS = {"16x4": ([4] * 16, 8, 96), "32x4": ([4] * 32, 8, 64), "664": ([6, 6, 4] * 4, 16, 48), "40": ([6, 5, 5, 6, 5, 5, 4, 4], 16, 48),
           "8x8": ([8] * 8, 16, 32), "655": ([6, 5, 5] * 4, 16, 48), "16x8": ([8] * 16, 16, 32), "664x2": ([6, 6, 4] * 8, 16, 48), "16x4w": ([4] * 16, 16, 32),
           "odd": ([3, 5, 7, 2], 8, 20)}


@pytest.mark.parametrize("kind", ["random", "few different", "equal"])
@pytest.mark.parametrize("R", [1, 100, 128, 129, 700])
@pytest.mark.parametrize("name", list(LAYOUTS))
def test_long_lists(name, R, kind):
    check(name, R, kind, [1023, 1024, 1025, 0, 60_001, 3, 4097, 30_000])


@pytest.mark.parametrize("threads", [64, 128, 256])
@pytest.mark.parametrize("R", [1, 100, 700])
@pytest.mark.parametrize("name", ["16x4", "32x4", "664", "40", "664x2", "odd"])
def test_near_codes_last(name, R, threads):
    check(name, R, "late", [4095, 4097, 8191, 8192, 8193, 16_385, 25_001, 50_000], threads)


def distances(codes, nbits, dsub, cb, z):
    """float64 distances of packed codes to z"""
    bits = np.unpackbits(codes, axis=1, bitorder="little")
    out, off, o, c0 = np.zeros(codes.shape[0]), 0, 0, 0
    for b, s in zip(nbits, dsub):
        c = cb[c0:c0 + (s << b)].reshape(1 << b, s).astype(np.float64)
        sub = bits[:, off:off + b].astype(np.int64) @ (1 << np.arange(b))
        out += ((c - z[o:o + s]) ** 2).sum(1)[sub]
        off, o, c0 = off + b, o + s, c0 + (s << b)
    return out


def check(name, R, kind, lens, threads=128):
    from paper_1812_09162_amd import binding as qb
    nbits, acc, d = LAYOUTS[name]
    rng = np.random.default_rng(R + len(name))
    B = sum(nbits)
    dsub = [d * b // B for b in nbits]
    dsub[0] += d - sum(dsub)
    n, K = sum(lens), len(lens)
    cb = rng.standard_normal(sum((1 << b) * s for b, s in zip(nbits, dsub))).astype(np.float32)
    coarse = (0.3 * rng.standard_normal((K, d))).astype(np.float32)
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    codes = rng.integers(0, 256, (n, (B + 7) // 8), dtype=np.uint8)
    if B % 8:
        codes[:, -1] &= (1 << (B % 8)) - 1
    if kind in ("few different", "equal"):
        codes = codes[rng.integers(0, 9, n) if kind == "few different" else np.zeros(n, dtype=np.int64)]
    ids = rng.permutation(n).astype(np.int32)
    q = rng.standard_normal((3, d)).astype(np.float32)
    probe = np.stack([rng.permutation(K) for _ in range(3)]).astype(np.int32)
    if kind == "late":
        for c in range(K):
            part = codes[off[c]:off[c + 1]]
            codes[off[c]:off[c + 1]] = part[np.argsort(-distances(part, nbits, dsub, cb, q[0] - coarse[c]), kind="stable")]
    dev = torch.device("cuda:0")
    idx = qb.PqIndex(d, nbits, dsub, torch.from_numpy(cb).to(dev), acc)
    args = [idx] + [torch.from_numpy(np.ascontiguousarray(x)).to(dev) for x in (coarse, off, codes, ids, q, probe)] + [400, R]
    qb.pq_set_option(qb.PQ_OPT_IVF_THREADS, threads)
    try:
        gi, gd = qb.ivf_adc_scan_topk(*args)
        qb.pq_set_option(qb.PQ_OPT_IVF_SHARED_LISTS, 2)
        si, sd = qb.ivf_adc_scan_topk(*args)
    finally:
        qb.pq_set_option(qb.PQ_OPT_IVF_SHARED_LISTS, 1)
        qb.pq_set_option(qb.PQ_OPT_IVF_THREADS, 128)
    torch.cuda.synchronize()
    assert torch.equal(gi, si) and torch.equal(gd, sd)
    for a in range(3):
        oi, od, _ = oracle.search_ivf(d, nbits, dsub, acc, cb, coarse, off, codes, ids, q[a], probe[a], 400, R)
        assert np.array_equal(gi[a].cpu().numpy(), oi) and np.array_equal(gd[a].cpu().numpy(), od), a
    idx.close()
