"""One pass over a list for up to sixteen pairs on the matrix cores (k_ivf_scan_mx), at the sizes where it can go
wrong: list starts of both parities, lists around one block of 64 codes and around the four waves' share, cells
with fewer pairs than columns and with several groups, bounds that admit nothing and everything.  Every result
is defined bit for bit, so it is compared with the scan of a block per pair, and a sample with the oracle."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def qb():
    from paper_1812_09162_amd import binding
    return binding


def problem(ds, lens, nq, nprobe, seed, identical=False, scale=1.0):
    rng = np.random.default_rng(seed)
    d, K, n = 16 * ds, len(lens), int(sum(lens))
    p = dict(d=d, nbits=[4] * 16, dsub=[ds] * 16, K=K)
    p["cb"] = (rng.standard_normal(256 * ds) * scale).astype(np.float32)
    p["coarse"] = rng.standard_normal((K, d)).astype(np.float32)
    p["off"] = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    p["codes"] = rng.integers(0, 256, (n, 8), dtype=np.uint8)
    if identical:
        p["codes"][:] = p["codes"][0]
    p["ids"] = rng.permutation(n).astype(np.int32)
    p["q"] = rng.standard_normal((nq, d)).astype(np.float32)
    p["probe"] = np.stack([rng.permutation(K)[:nprobe] for _ in range(nq)]).astype(np.int32)
    return p


def run_both(qb, p, R, sample=3):
    dev = torch.device("cuda:0")
    idx = qb.PqIndex(p["d"], p["nbits"], p["dsub"], torch.from_numpy(p["cb"]).to(dev), 8)
    args = [idx] + [torch.from_numpy(p[k]).to(dev) for k in ("coarse", "off", "codes", "ids", "q", "probe")] + [400, R]
    out = []
    for opt in (0, 2):
        qb.pq_set_option(qb.PQ_OPT_IVF_SHARED_LISTS, opt)
        try:
            out.append(qb.ivf_adc_scan_topk(*args))
            torch.cuda.synchronize()
        finally:
            qb.pq_set_option(qb.PQ_OPT_IVF_SHARED_LISTS, 1)
    (i0, d0), (i1, d1) = out
    assert torch.equal(i0, i1) and torch.equal(d0, d1)
    for q in range(min(sample, p["q"].shape[0])):
        oi, od, _ = oracle.search_ivf(p["d"], p["nbits"], p["dsub"], 8, p["cb"], p["coarse"], p["off"], p["codes"],
                                      p["ids"], p["q"][q], p["probe"][q], 400, R)
        assert np.array_equal(i1[q].cpu().numpy(), oi) and np.array_equal(d1[q].cpu().numpy(), od)
    idx.close()


@pytest.mark.parametrize("ds", [4, 6, 8])
@pytest.mark.parametrize("nq", [1, 15, 16, 17, 40])  # pairs per cell: around one group of sixteen and three of them
def test_list_lengths(qb, ds, nq):
    lens = [1, 2, 3, 63, 64, 65, 127, 128, 129, 0, 255, 256, 257, 319, 320, 321, 1000, 1537, 4096, 77]
    run_both(qb, problem(ds, lens, nq, len(lens), 100 * ds + nq), 100)


@pytest.mark.parametrize("R", [1, 10, 1000, 2000])
@pytest.mark.parametrize("scale", [0.05, 1.0, 20.0])  # lists that are skipped, ordinary ones, entries that saturate
def test_bounds(qb, R, scale):
    run_both(qb, problem(6, [700, 701, 333, 2049, 90, 5000, 12, 1200], 33, 6, 7 + R, scale=scale), R)


@pytest.mark.parametrize("R", [1, 100])
def test_every_code_within_the_bound(qb, R):
    # equal codes: one distance per list, every one of them is queued and the slot lists overflow
    run_both(qb, problem(6, [1500, 1501, 3000, 64], 20, 4, 5, identical=True), R)
