"""Calls that run beside others on several streams, each with its own workspace and outputs, against the same call alone: short
lists scanned by the quantizer's blocks, pilots counted four queries to a block, the tightening search and inverted lists long enough
that their slots are cut back.  Every result is defined bit for bit."""
import numpy as np
import pytest
import torch

from test_gpu_ivf_shared import problem, qb  # noqa: F401  (the fixture)

pytestmark = pytest.mark.gpu


def beside_each_other(calls, rounds=6):
    """calls[i](stream's own copies) -> tensors; every call on every stream at once, several times"""
    alone = [[x.clone() for x in c()] for c in calls]
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in range(4)]
    out = []
    for r in range(rounds):
        for i, st in enumerate(streams):
            with torch.cuda.stream(st):
                for k in range(len(calls)):
                    j = (i + k + r) % len(calls)
                    out.append((j, calls[j]()))
    torch.cuda.synchronize()
    for j, got in out:
        for a, b in zip(got, alone[j]):
            assert torch.equal(a.contiguous().view(torch.uint8), b.contiguous().view(torch.uint8)), j


@pytest.mark.parametrize("name,nbits,acc", [("16x4", [4] * 16, 8), ("664", [6, 6, 4] * 4, 16), ("16x8", [8] * 16, 16)])
def test_exhaustive_calls(qb, name, nbits, acc):  # noqa: F811
    d, dev, rng = 96, torch.device("cuda:0"), np.random.default_rng(acc + len(nbits))
    dsub = [d * b // sum(nbits) for b in nbits]
    dsub[0] += d - sum(dsub)
    cb = torch.from_numpy(rng.standard_normal(sum((1 << b) * s for b, s in zip(nbits, dsub))).astype(np.float32)).to(dev)
    idx = qb.PqIndex(d, nbits, dsub, cb, acc)
    codes = torch.from_numpy(rng.integers(0, 256, (300_001, (sum(nbits) + 7) // 8), dtype=np.uint8)).to(dev)
    q = torch.from_numpy(rng.standard_normal((300, d)).astype(np.float32)).to(dev)
    tables = qb.pq_compute_tables(idx, q)
    beside_each_other([lambda: qb.pq_search_topk(idx, q[:1], codes[:100_000], 400, 100),
                       lambda: qb.pq_search_topk(idx, q[3:20], codes[:65_537], 400, 10),
                       lambda: qb.pq_search_topk(idx, q[20:22], codes, 400, 100),
                       lambda: qb.pq_quantize_tables(idx, tables, codes[:70_000], 400, 100)])
    idx.close()


def test_inverted_lists(qb):  # noqa: F811
    p = problem(6, [30_000, 9000, 12, 4097, 700, 20_001], 40, 5, 77)
    dev = torch.device("cuda:0")
    idx = qb.PqIndex(p["d"], p["nbits"], p["dsub"], torch.from_numpy(p["cb"]).to(dev), 8)
    lists = [idx] + [torch.from_numpy(p[k]).to(dev) for k in ("coarse", "off", "codes", "ids")]
    q, probe = torch.from_numpy(p["q"]).to(dev), torch.from_numpy(p["probe"]).to(dev)
    beside_each_other([lambda: qb.ivf_adc_scan_topk_tightening(*lists, q, probe, 400, 100),
                       lambda: qb.ivf_adc_scan_topk_tightening(*lists, q[:3].contiguous(), probe[:3].contiguous(), 400, 200),
                       lambda: qb.ivf_adc_scan_topk(*lists, q[:5].contiguous(), probe[:5].contiguous(), 400, 100),
                       lambda: qb.ivf_adc_scan_topk(*lists, q, probe, 400, 10)])
    idx.close()
