"""GPU parity of the batched scan on the matrix cores: every query of a batch must give, byte for
byte, what it gives alone (one query per call takes a different kernel), and a sample must match
the CPU oracle.  Sizes sit at the edges of the 512- and 2048-code chunks, of the 32-query tiles and
of the block that picks the results."""
import threading

import numpy as np
import pytest
import torch

import oracle
from harness import synth
from paper_1812_09162_amd import binding as qb

pytestmark = pytest.mark.gpu

LAYOUTS = {
    "16x4": ([4] * 16, 8), "16x4u16": ([4] * 16, 16), "32x4": ([4] * 32, 8),
    "c3": ([6, 5, 5, 6, 5, 5, 4, 4], 16), "c3u8": ([6, 5, 5, 6, 5, 5, 4, 4], 8), "5x8": ([5] * 8, 16), "40six": ([6, 5, 6, 5, 6, 4, 4, 4], 16),
    "664": ([6, 6, 4] * 4, 16), "655": ([6, 5, 5] * 4, 16), "664u8": ([6, 6, 4] * 4, 8),
    "6to4": ([6] * 8 + [4] * 4, 16),  # as many steps of each kind as {6,6,4} x 4, fields elsewhere
    "odd64": ([4, 5, 6, 5, 4, 6, 6, 5, 5, 4, 6, 5], 16),
    "664x2": ([6, 6, 4] * 8, 16), "655x2": ([6, 5, 5] * 8, 16), "mixed128": ([4, 6, 6, 5, 5, 6, 4, 6, 6, 5, 5, 6] * 2, 16),
}


def _make(name, n, nq, seed, data="aniso_gauss", d=96):
    nbits, acc = LAYOUTS[name]
    lay = synth.make_layout(d, nbits, acc)
    g = torch.Generator().manual_seed(seed)
    x = synth.GENERATORS[data](4096, d, seed)
    cbs, o = [], 0
    for k, s in zip(lay.ksub, lay.dsub):
        cbs.append(x[torch.randperm(4096, generator=g)[:k], o:o + s].reshape(-1))
        o += s
    cb = torch.cat(cbs).contiguous()
    sub = torch.stack([torch.randint(0, k, (n,), generator=g) for k in lay.ksub], 1).to(torch.uint8)
    codes = synth.pack_codes(sub, lay)
    queries = synth.GENERATORS[data](nq, d, seed + 1)
    idx = qb.PqIndex(d, lay.nbits, lay.dsub, cb.cuda(), acc)
    return lay, cb, codes, queries, idx


def _matrix(idx, nq, n, R):
    """the call is one of the matrix cores' (whose sizes pq_search_form knows)"""
    assert qb.pq_search_form(idx, nq, n, R) == qb.PQ_SCAN_MATRIX
    return True


def _check(lay, cb, codes, queries, idx, R, sample=2, t=400):
    c, z = codes.cuda(), queries.cuda()
    got = qb.pq_search_topk(idx, z, c, t, R)
    for q in range(z.shape[0]):
        one = qb.pq_search_topk(idx, z[q:q + 1], c, t, R)
        for a, b in zip(got, one):
            assert torch.equal(a[q].view(torch.uint8), b[0].view(torch.uint8)), q
    for q in range(0, z.shape[0], max(1, z.shape[0] // sample))[:sample] if sample else []:
        oi, ok, od = oracle.search(lay.d, lay.nbits, lay.dsub, lay.acc_bits, cb.numpy(), queries[q].numpy(),
                                   codes.numpy(), t, R)
        assert np.array_equal(got[0][q].cpu().numpy(), oi)
        assert np.array_equal(got[1][q].cpu().numpy().astype(np.uint16), ok)
        assert np.array_equal(got[2][q].cpu().numpy(), od)
    return got


# (The matrix cores take a batch from some 800,000 codes times passes of four queries on, irregular
# layouts from 6,000,000 on, and from 1,000 / 8,000 codes per result on, and more where that does not
# pay: _matrix() asks.  Smaller calls are look-ups, which also have to agree with the single query.)
@pytest.mark.parametrize("name", list(LAYOUTS))
@pytest.mark.parametrize("n,nq,R", [(262_144, 97, 32), (131_583, 225, 1), (300_033, 84, 33)])
def test_batch_equals_single(name, n, nq, R):
    _check(*_make(name, n, nq, 3 + len(name)), R, sample=1)


# per layout: codes, queries, results at which it is the matrix cores' turn (40-bit codes and 128-bit ones of
# other fields have the narrowest range)
MATRIX_SIZES = {
    "16x4": (262_144, 97, 32), "16x4u16": (262_144, 97, 32), "32x4": (131_583, 225, 1), "c3": (1_600_001, 17, 100),
    "c3u8": (1_607_680, 16, 100), "5x8": (1_600_513, 18, 100), "40six": (1_600_513, 18, 100),
    "664": (300_033, 84, 33), "655": (262_144, 97, 32),
    "664u8": (300_033, 84, 33), "6to4": (800_001, 33, 33), "odd64": (800_513, 61, 50), "664x2": (131_583, 225, 1),
    "655x2": (300_033, 84, 33), "mixed128": (800_100, 40, 33),
}


@pytest.mark.parametrize("name", list(LAYOUTS))
def test_matrix_form_equals_single(name):
    n, nq, R = MATRIX_SIZES[name]
    lay, cb, codes, queries, idx = _make(name, n, nq, 30 + len(name))
    assert _matrix(idx, nq, n, R)
    _check(lay, cb, codes, queries, idx, R, sample=1)


@pytest.mark.parametrize("name", ["c3", "664", "16x4u16"])
def test_matrix_form_single_best(name):
    lay, cb, codes, queries, idx = _make(name, 1_600_003, 17, 40)
    assert _matrix(idx, 17, 1_600_003, 1)
    _check(lay, cb, codes, queries, idx, 1, sample=1)


@pytest.mark.parametrize("n", [200_704, 200_703, 200_705, 2048 * 100 - 1, 2048 * 100, 2048 * 100 + 513])
@pytest.mark.parametrize("nq", [40, 65, 97])
def test_matrix_form_chunk_and_tile_edges(n, nq):
    lay, cb, codes, queries, idx = _make("16x4", n, nq, n + nq)
    assert _matrix(idx, nq, n, 10)
    _check(lay, cb, codes, queries, idx, 10, sample=1)


def test_which_form():
    """the lines the rule draws: what is taken, and what stays with the look-ups (or went back to them)"""
    idx = {name: _make(name, 64, 1, 1)[4] for name in LAYOUTS}
    yes = [("16x4", 5, 10_000_000, 100), ("16x4", 9, 10_000_000, 1000), ("16x4", 256, 100_000, 10), ("16x4", 48, 110_000, 100), ("32x4", 100, 50_000, 1),
           ("c3", 32, 10_000_000, 100), ("c3", 32, 1_000_000, 100), ("c3", 32, 1_600_000, 64), ("664", 5, 4_000_000, 100),
           ("664", 32, 10_000_000, 100), ("664x2", 5, 4_000_000, 100), ("odd64", 13, 4_000_000, 100), ("5x8", 8, 4_000_000, 100),
           ("mixed128", 24, 1_000_000, 100), ("32x4", 8, 10_000_000, 500), ("16x4u16", 13, 4_000_000, 500)]
    no = [("16x4", 4, 10_000_000, 100), ("16x4", 8, 10_000_000, 1000), ("16x4", 32, 100_000, 10), ("32x4", 8, 10_000_000, 1000),
          ("c3", 64, 2_000_000, 64), ("c3", 32, 800_000, 1), ("c3", 64, 8_000_000, 1000), ("c3", 64, 1_000_000, 100),
          ("664", 5, 4_000_000, 1), ("664", 8, 10_000_000, 500), ("664u8", 100, 800_000, 1), ("655x2", 8, 4_000_000, 250),
          ("odd64", 12, 4_000_000, 100), ("odd64", 60, 400_000, 32), ("5x8", 64, 1_600_000, 1), ("5x8", 7, 4_000_000, 100),
          ("mixed128", 100, 4_000_000, 100), ("mixed128", 16, 1_000_000, 100), ("16x4u16", 8, 4_000_000, 500), ("664", 64, 4_000_000, 10)]
    stage_yes = [("16x4", 5, 4_000_000, 100), ("16x4", 1000, 1_000_003, 100), ("16x4", 32, 1_000_000, 10), ("32x4", 12, 4_000_000, 1),
                 ("664", 16, 4_000_000, 100), ("664x2", 24, 8_000_000, 250), ("c3", 16, 4_000_000, 100), ("odd64", 32, 2_000_000, 100)]
    stage_no = [("16x4", 8, 400_000, 100), ("16x4", 32, 400_000, 10), ("16x4", 256, 4_000_000, 1), ("664", 8, 4_000_000, 100),
                ("664x2", 12, 8_000_000, 250), ("c3", 8, 4_000_000, 100), ("odd64", 16, 1_600_000, 100), ("mixed128", 64, 1_600_000, 64)]
    for name, nq, n, R in stage_yes:
        assert qb.pq_scan_form(idx[name], nq, n, R) == qb.PQ_SCAN_MATRIX, (name, nq, n, R)
    for name, nq, n, R in stage_no:
        assert qb.pq_scan_form(idx[name], nq, n, R) == qb.PQ_SCAN_LOOKUP, (name, nq, n, R)
    for name, nq, n, R in yes:
        assert qb.pq_search_form(idx[name], nq, n, R) == qb.PQ_SCAN_MATRIX, (name, nq, n, R)
    for name, nq, n, R in no:
        assert qb.pq_search_form(idx[name], nq, n, R) == qb.PQ_SCAN_LOOKUP, (name, nq, n, R)


@pytest.mark.parametrize("n", [16_384, 16_895, 16_896, 16_897, 2048 * 32 - 1, 2048 * 32 + 513])
@pytest.mark.parametrize("nq", [200, 225, 257])
def test_chunk_and_tile_edges(n, nq):
    _check(*_make("16x4", n, nq, n + nq), 10, sample=1)


@pytest.mark.parametrize("name,n,R", [(s, n, R) for s, n in [("16x4", 600_001), ("32x4", 600_001), ("16x4u16", 600_001)]
                                      for R in [1, 128, 129, 256, 257, 600]] + [("c3", 2_500_003, 300), ("664", 2_500_003, 129)])
def test_result_lengths(name, n, R):
    _check(*_make(name, n, 12, R), R, sample=1)


def test_small_blocks_and_large_chunks():
    """more than 512 queries (small picking blocks); 16 groups per lane and chunk"""
    _check(*_make("16x4", 100_007, 513, 8), 100, sample=1)
    lay, cb, codes, queries, idx = _make("16x4", 4_200_003, 40, 9)
    _check(lay, cb, codes, queries[:34], idx, 100, sample=0)
    _check(lay, cb, codes, queries[:6], idx, 1, sample=0)  # (groups of more than 64 codes: little workspace)


@pytest.mark.parametrize("name,n,nq,R", [("16x4", 100_000, 130, 100), ("c3", 262_144, 130, 32), ("16x4", 200_001, 40, 100),
                                         ("664", 262_144, 100, 32), ("c3", 1_600_001, 16, 100)])
@pytest.mark.parametrize("distinct", [1, 7, 300])
def test_equal_codes(name, n, nq, R, distinct):
    """crowds of equal keys: list overflow, segments, exact selection"""
    lay, cb, codes, queries, idx = _make(name, n, nq, 11)
    assert nq == 130 or _matrix(idx, nq, n, R)
    g = torch.Generator().manual_seed(4)
    codes = codes[torch.randint(0, distinct, (n,), generator=g)].contiguous()
    _check(lay, cb, codes, queries, idx, R, sample=1)


@pytest.mark.parametrize("n", [110_000, 220_000])
def test_integer_data_and_calibration_at_the_end(n):
    """integer tables (many ties); the first codes the best ones (everything else saturates) and the worst ones"""
    lay, cb, codes, queries, idx = _make("16x4", n, 40, 12, "gamma_ints", 128)
    assert n == 110_000 or _matrix(idx, 40, n, 100)
    _check(lay, cb, codes, queries, idx, 100)
    ids = qb.pq_search_topk(idx, queries[:1].cuda(), codes.cuda(), 400, 2000)[0][0].cpu().long()
    rest = torch.ones(n, dtype=torch.bool)
    rest[ids] = False
    best_first = torch.cat([codes[ids], codes[rest]])
    _check(lay, cb, best_first.contiguous(), queries, idx, 100, sample=1)
    _check(lay, cb, best_first.flip(0).contiguous(), queries, idx, 100, sample=1)


@pytest.mark.parametrize("R", [1, 2, 3])
@pytest.mark.parametrize("nq,n", [(5, 1_000_003), (64, 200_001)])
def test_saturated_result(nq, n, R):
    """The result is saturated, and so is every other code: of all of them the lowest ids are the answer,
    also where these have larger sums than the best code's group (levels of entries are not clamped)."""
    lay = synth.make_layout(16, [4] * 16, 8)
    cb = torch.arange(16, dtype=torch.float32).repeat(16)
    sub = torch.zeros((n, 16), dtype=torch.uint8)
    sub[:, :3] = 2
    sub[300] = 0
    sub[300, 0] = 1
    codes, queries = synth.pack_codes(sub, lay), torch.zeros(nq, 16)
    idx = qb.PqIndex(16, lay.nbits, lay.dsub, cb.cuda(), 8)
    assert _matrix(idx, nq, n, R)
    got = _check(lay, cb, codes, queries, idx, R, sample=1)
    if R == 1:
        assert got[0].eq(0).all() and got[1].cpu().numpy().min() == 255


@pytest.mark.parametrize("name,n,nq", [("c3", 262_144, 97), ("664", 262_144, 97), ("16x4u16", 262_144, 97), ("c3", 1_600_003, 18)])
def test_saturated_best_code(name, n, nq):
    """Queries far from all centroids, the best code of each among the calibration codes: fp32 sums against
    the fp64 sum of the entries leave it, for some of them, just above the top of the range, with all others."""
    lay, cb, codes, queries, _ = _make(name, n, nq, 21)
    queries = queries + 150.0
    o = dims = 0
    best = torch.zeros(nq, codes.shape[0])
    sub = oracle.unpack(lay.nbits, codes.numpy())
    for j, (k, s) in enumerate(zip(lay.ksub, lay.dsub)):
        c = cb[o:o + k * s].reshape(k, s).double()
        t = (queries[:, None, dims:dims + s].double() - c[None]).square().sum(2)
        best += t[:, torch.from_numpy(sub[:, j].astype(np.int64))].float()
        o, dims = o + k * s, dims + s
    codes[300:300 + nq] = codes[best.argmin(1)].clone()
    idx = qb.PqIndex(lay.d, lay.nbits, lay.dsub, cb.cuda(), lay.acc_bits)
    assert (name == "c3" and n == 262_144) or _matrix(idx, nq, n, 1)
    _check(lay, cb, codes, queries, idx, 1)


@pytest.mark.parametrize("n", [90_000, 1_000_003])
def test_stage_calls_and_bounds(n):
    """the scan call with the quantizer's bound, an unknown one, and one below which few codes lie"""
    lay, cb, codes, queries, idx = _make("16x4", n, 40, 13)
    assert n == 90_000 or qb.pq_scan_form(idx, 40, n, 50) == qb.PQ_SCAN_MATRIX
    c, z = codes.cuda(), queries.cuda()
    tables = qb.pq_compute_tables(idx, z)
    qt, qp = qb.pq_quantize_tables(idx, tables, c, 400, 50)
    want = qb.pq_search_topk(idx, z, c, 400, 50)
    for bound in (None, qb.PQ_KEY_BOUND_UNKNOWN, 40):
        p = qp.clone()
        if bound is not None:
            p.view(torch.int32).view(40, 6)[:, 5] = bound if bound < 2 ** 31 else bound - 2 ** 32
        got = qb.pq_adc_scan_topk(idx, qt, p, c, 50)
        for q in range(40):
            one = qb.pq_adc_scan_topk(idx, qt[q:q + 1].contiguous(), p[q:q + 1].contiguous(), c, 50)
            for a, b, w in zip(got, one, want):
                assert torch.equal(a[q], b[0])
                if bound != 40:
                    assert torch.equal(a[q], w[q])


def test_option_set_by_another_thread():
    """PQ_OPT_SHARED_PASSES changes no result, whenever it is set: a call prepares its tables for the scan
    that it then runs"""
    lay, cb, codes, queries, idx = _make("16x4", 400_000, 9, 14)
    c, z = codes.cuda(), queries.cuda()
    assert _matrix(idx, 9, 400_000, 20)
    want = qb.pq_search_topk(idx, z, c, 400, 20)
    done = threading.Event()

    def toggle():
        while not done.is_set():
            qb.pq_set_option(qb.PQ_OPT_SHARED_PASSES, 0)
            qb.pq_set_option(qb.PQ_OPT_SHARED_PASSES, 1)

    thread = threading.Thread(target=toggle)
    thread.start()
    try:
        for _ in range(300):
            got = qb.pq_search_topk(idx, z, c, 400, 20)
            assert all(torch.equal(a.view(torch.uint8), b.view(torch.uint8)) for a, b in zip(got, want))
    finally:
        done.set()
        thread.join()
        qb.pq_set_option(qb.PQ_OPT_SHARED_PASSES, 1)
