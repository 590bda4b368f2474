"""The tightening search's kernel for 16 x 4 bits over equal sub-spaces, at the sizes where it can go wrong: lists around a
block's 512 threads, a round of 2048 codes and a segment of 4096, lists that fill the candidate buffer (once by their first
codes, or with one distance throughout), empty lists and invalid cells between others, more than a chunk of 64 probes, skipped
lists, results around one, two and four places per lane.  Compared with the oracle, bit for bit."""
import numpy as np
import pytest
import torch

import oracle
from test_gpu_ivf_shared import problem, qb  # noqa: F401  (the fixture)

pytestmark = pytest.mark.gpu


def run(qb, p, R):
    dev = torch.device("cuda:0")
    idx = qb.PqIndex(p["d"], p["nbits"], p["dsub"], torch.from_numpy(p["cb"]).to(dev), 8)
    args = [idx] + [torch.from_numpy(p[k]).to(dev) for k in ("coarse", "off", "codes", "ids", "q", "probe")] + [400, R]
    ids, dist = qb.ivf_adc_scan_topk_tightening(*args)
    torch.cuda.synchronize()
    probe = np.where(p["probe"] < p["K"], p["probe"], -1)  # (the oracle takes cells of the index only)
    for q in range(p["q"].shape[0]):
        oi, od, _, _ = oracle.search_ivf_tightening(p["d"], p["nbits"], p["dsub"], 8, p["cb"], p["coarse"], p["off"], p["codes"],
                                                    p["ids"], p["q"][q], probe[q], 400, R)
        assert np.array_equal(ids[q].cpu().numpy(), oi), q
        assert np.array_equal(dist[q].cpu().numpy(), od), q
    idx.close()


LENS = [1, 2, 0, 63, 64, 65, 0, 0, 511, 512, 513, 1537, 2047, 2048, 2049, 4095, 4096, 4097, 0, 8200, 77, 300]


@pytest.mark.parametrize("ds", [4, 6, 8])
@pytest.mark.parametrize("R", [1, 64, 65, 100, 128, 129, 256, 257])
def test_list_lengths(qb, ds, R):  # noqa: F811
    p = problem(ds, LENS, 5, len(LENS), 100 * ds + R)
    p["probe"][1, ::3] = -1
    p["probe"][2, 1::4] = len(LENS)
    if R <= 256:
        p["probe"][3, :] = p["probe"][3, 0]  # one list again and again: equal words, equal ids
    run(qb, p, R)


@pytest.mark.parametrize("R", [1, 100, 200])
@pytest.mark.parametrize("scale", [0.05, 1.0, 20.0])  # lists that are skipped, ordinary ones, entries that saturate
def test_many_probes(qb, R, scale):  # noqa: F811
    rng = np.random.default_rng(R)
    lens = [int(x) for x in rng.integers(0, 40, 200)]
    run(qb, problem(6, lens, 4, 150, 17 + R, scale=scale), R)


@pytest.mark.parametrize("R", [1, 100, 256])
@pytest.mark.parametrize("kind", ["long", "few different", "equal"])
def test_candidate_buffer_runs_full(qb, R, kind):  # noqa: F811
    p = problem(6, [300, 30_000, 9_000, 20_001, 5], 3, 5, 23 + R, identical=kind == "equal")
    if kind == "few different":
        p["codes"][:] = p["codes"][np.arange(p["codes"].shape[0]) % 7]
    p["probe"][0] = [1, 0, 2, 3, 4]
    p["probe"][1] = [0, 1, 3, 2, 4]
    run(qb, p, R)


@pytest.mark.parametrize("R", [1, 100, 256])
def test_late_segments_overflow(qb, R):  # noqa: F811
    # a list of many segments, the first query's far codes first: the fill level left by the ones before is what an overflow goes back to
    p = problem(6, [700, 41_000, 12_289, 8192, 300], 3, 5, 31 + R)
    for c in range(p["K"]):
        lo, hi = p["off"][c], p["off"][c + 1]
        z = (p["q"][0] - p["coarse"][c]).reshape(16, 1, 6)
        tab = ((z - p["cb"].reshape(16, 16, 6)) ** 2).sum(2)
        codes = p["codes"][lo:hi]
        nib = np.stack([codes & 15, codes >> 4], axis=2).reshape(-1, 16)
        p["codes"][lo:hi] = codes[np.argsort(-tab[np.arange(16), nib].sum(1), kind="stable")]
    p["probe"][:] = [0, 1, 2, 3, 4]
    run(qb, p, R)
