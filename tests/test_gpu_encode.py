"""GPU parity of pq_encode (through the C ABI) against the CPU oracle: packed codes byte for byte,
on all layouts, ragged counts, with and without the residual shift, and at a size that spans many
blocks; plus the chain encode -> search on the GPU against the oracle's own chain."""
import numpy as np
import pytest
import torch

import oracle
from harness import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def qb():
    from paper_1812_09162_amd import binding
    binding.load()
    return binding


def dev():
    return torch.device("cuda:0")


def layout_and_codebooks(d, nbits, seed, integer=False):
    lay = synth.make_layout(d, nbits, 16)
    rng = np.random.default_rng(seed)
    ncb = sum((1 << b) * s for b, s in zip(lay.nbits, lay.dsub))
    cb = (rng.integers(-6, 7, ncb) if integer else rng.normal(size=ncb)).astype(np.float32)
    return lay, cb


@pytest.mark.parametrize("d,nbits", [
    (128, [4] * 16), (96, [4] * 16), (128, [4] * 32), (128, synth.C3_BITS), (128, [8] * 8),
    (128, [6, 6, 4] * 8), (13, [3, 7, 1, 2]), (64, [8] * 16), (256, [4] * 16), (15, [5, 5, 5]),
])
@pytest.mark.parametrize("n", [1, 63, 64, 65, 127, 129, 1000])
def test_encode_bit_exact(qb, d, nbits, n):
    lay, cb = layout_and_codebooks(d, nbits, seed=len(nbits) + d)
    rng = np.random.default_rng(n)
    x = rng.normal(size=(n, d)).astype(np.float32)
    idx = qb.PqIndex(lay.d, lay.nbits, lay.dsub, torch.from_numpy(cb).to(dev()), 16)
    got = qb.pq_encode(idx, torch.from_numpy(x).to(dev())).cpu().numpy()
    assert np.array_equal(got, oracle.encode(d, lay.nbits, lay.dsub, cb, x))
    idx.close()


def test_encode_ties_go_to_the_lowest_index(qb):
    lay, cb = layout_and_codebooks(24, [4, 5, 3, 6], seed=3, integer=True)   # duplicate centroids abound
    rng = np.random.default_rng(4)
    x = rng.integers(-6, 7, (777, 24)).astype(np.float32)
    idx = qb.PqIndex(lay.d, lay.nbits, lay.dsub, torch.from_numpy(cb).to(dev()), 16)
    got = qb.pq_encode(idx, torch.from_numpy(x).to(dev())).cpu().numpy()
    assert np.array_equal(got, oracle.encode(24, lay.nbits, lay.dsub, cb, x))
    idx.close()


def test_encode_residuals(qb):
    lay, cb = layout_and_codebooks(96, [4] * 16, seed=8)
    rng = np.random.default_rng(9)
    n, K = 5000, 37
    x = rng.normal(size=(n, 96)).astype(np.float32)
    coarse = rng.normal(size=(K, 96)).astype(np.float32)
    ids = rng.integers(0, K, n).astype(np.int32)
    idx = qb.PqIndex(lay.d, lay.nbits, lay.dsub, torch.from_numpy(cb).to(dev()), 8)
    got = qb.pq_encode(idx, torch.from_numpy(x).to(dev()), torch.from_numpy(coarse).to(dev()),
                       torch.from_numpy(ids).to(dev())).cpu().numpy()
    assert np.array_equal(got, oracle.encode(96, lay.nbits, lay.dsub, cb, x, coarse[ids]))
    idx.close()


def test_encode_then_search_matches_the_oracle_chain(qb):
    pr = synth.build(synth.scaled("C3", n=20_000, nq=3))
    lay = pr.layout
    rng = np.random.default_rng(12)
    x = np.minimum(255, np.floor(rng.gamma(0.5, 7.27, (20_000, lay.d)))).astype(np.float32)
    idx = qb.PqIndex(lay.d, lay.nbits, lay.dsub, pr.codebooks.to(dev()), lay.acc_bits)
    codes = qb.pq_encode(idx, torch.from_numpy(x).to(dev()))
    ocodes = oracle.encode(lay.d, lay.nbits, lay.dsub, pr.codebooks.numpy(), x)
    assert np.array_equal(codes.cpu().numpy(), ocodes)
    ids, keys, dist = qb.pq_search_topk(idx, pr.queries.to(dev()), codes, 400, 50)
    torch.cuda.synchronize()
    for q in range(pr.queries.shape[0]):
        oi, ok, od = oracle.search(lay.d, lay.nbits, lay.dsub, lay.acc_bits, pr.codebooks.numpy(),
                                   pr.queries[q].numpy(), ocodes, 400, 50)
        assert np.array_equal(ids[q].cpu().numpy(), oi)
        assert np.array_equal(dist[q].cpu().numpy(), od)
    idx.close()


def test_encode_large_sampled(qb):
    """2,000,003 vectors of the C1 shape: every code must decode to a nearest centroid; a sample is
    compared with the oracle."""
    cfg = synth.scaled("C1", n=1000, nq=1)
    pr = synth.build(cfg)
    lay = pr.layout
    g = torch.Generator(device=dev()).manual_seed(77)
    n = 2_000_003
    x = torch.randn((n, lay.d), generator=g, device=dev(), dtype=torch.float32)
    idx = qb.PqIndex(lay.d, lay.nbits, lay.dsub, pr.codebooks.to(dev()), lay.acc_bits)
    codes = qb.pq_encode(idx, x)
    torch.cuda.synchronize()
    sel = np.r_[0:300, n // 2:n // 2 + 300, n - 300:n]
    want = oracle.encode(lay.d, lay.nbits, lay.dsub, pr.codebooks.numpy(), x[sel].cpu().numpy())
    assert np.array_equal(codes[sel].cpu().numpy(), want)
    idx.close()


def test_encode_errors(qb):
    lay, cb = layout_and_codebooks(16, [4] * 4, seed=1)
    idx = qb.PqIndex(lay.d, lay.nbits, lay.dsub, torch.from_numpy(cb).to(dev()), 8)
    x = torch.zeros((4, 16), dtype=torch.float32, device=dev())
    rc = qb.load().pq_encode(idx.handle, x.data_ptr(), 4, x.data_ptr(), None, x.data_ptr(), None)
    assert rc == qb.PQ_EINVAL
    assert qb.pq_encode(idx, x[:0]).shape == (0, 2)
    idx.close()


@pytest.mark.parametrize("d,nbits", [(96, [4] * 16), (128, [4] * 32), (64, [8] * 16), (36, [2, 3, 4, 6] * 2), (132, [4] * 32)])
@pytest.mark.parametrize("scale", [1.0, 1e-21, 1e-12, 1e18])
def test_encode_near_ties(qb, d, nbits, scale):
    """Vectors half way between two centroids of every sub-space, and a few units in the last place from
    there; duplicate centroids; data of any scale (the terms' squares underflow, or their sums overflow)."""
    lay = synth.make_layout(d, nbits, 16)
    rng = np.random.default_rng(d)
    parts, mids = [], []
    for b, s in zip(lay.nbits, lay.dsub):
        c = rng.normal(size=(1 << b, s)).astype(np.float32)
        c[-1] = c[0]
        parts.append(c)
        a, o = rng.integers(0, 1 << b, 600), rng.integers(0, 1 << b, 600)
        mids.append(((c[a].astype(np.float64) + c[o]) / 2).astype(np.float32))
    x = np.concatenate(mids, axis=1)
    x[200:] = np.nextafter(x[200:], np.float32(np.inf))
    x[400:] = np.nextafter(x[400:], np.float32(np.inf))
    cb = np.concatenate([p.reshape(-1) for p in parts]) * np.float32(scale)
    x = (x * np.float32(scale)).astype(np.float32)
    idx = qb.PqIndex(lay.d, lay.nbits, lay.dsub, torch.from_numpy(cb).to(dev()), 16)
    want = oracle.encode(d, lay.nbits, lay.dsub, cb, x)
    assert np.array_equal(qb.pq_encode(idx, torch.from_numpy(x).to(dev())).cpu().numpy(), want)
    # vectors and codes at addresses that allow no wide access
    flat = torch.empty(x.size + 1, device=dev())
    flat[1:] = torch.from_numpy(x.reshape(-1)).to(dev())
    room = torch.empty(want.size + 1, dtype=torch.uint8, device=dev())
    got = room[1:].view(want.shape)
    qb.pq_encode(idx, flat[1:].view(x.shape), codes=got)
    assert np.array_equal(got.cpu().numpy(), want)
    idx.close()


@pytest.mark.parametrize("d,nbits,n", [
    # the expanded form, which long lists take (256 vectors per table entry) ...
    (96, [4] * 16, 65_536 + 1), (96, [4] * 16, 262_144 + 129), (128, [4] * 16, 262_144 + 65), (128, [6, 6, 4] * 8, 300_001),
    (36, [4] * 6, 30_000), (20, [4] * 4, 20_001), (28, [5] * 4, 40_000), (132, [4] * 32, 262_144 + 65),
    # ... and short ones with eight dimensions
    (128, [4] * 16, 600), (16, [5] * 2, 63),
    # term by term, tiles requested ahead (d = 128) and not
    (128, [8] * 8, 262_144 + 65), (96, [8] * 8, 262_144 + 65), (128, [4] * 32, 262_144 + 1),
])
@pytest.mark.parametrize("shift", [False, True])
def test_encode_forms_and_second_tiles(qb, d, nbits, n, shift):
    """Near ties as above in every form of the kernel, in lists long enough that a block encodes a second
    and a third tile (4096 blocks of 64 vectors), the last one partly filled."""
    lay = synth.make_layout(d, nbits, 16)
    rng = np.random.default_rng(n)
    parts, mids = [], []
    for b, s in zip(lay.nbits, lay.dsub):
        c = rng.normal(size=(1 << b, s)).astype(np.float32)
        c[-1] = c[0]
        parts.append(c)
        a, o = rng.integers(0, 1 << b, 601), rng.integers(0, 1 << b, 601)
        mids.append(((c[a].astype(np.float64) + c[o]) / 2).astype(np.float32))
    x = np.concatenate(mids, axis=1)
    x[300:] = np.nextafter(x[300:], np.float32(np.inf))
    x[450:] = rng.normal(size=x[450:].shape)
    cb = np.concatenate([p.reshape(-1) for p in parts])
    rows = rng.integers(-4, 5, size=(7, d)).astype(np.float32)
    ids = rng.integers(0, 7, size=601).astype(np.int32)
    if shift:
        x = x + rows[ids]
    want = oracle.encode(d, lay.nbits, lay.dsub, cb, x, rows[ids] if shift else None)
    pick = torch.arange(n, device=dev()) % 601
    idx = qb.PqIndex(lay.d, lay.nbits, lay.dsub, torch.from_numpy(cb).to(dev()), 16)
    xs = torch.from_numpy(x).to(dev())[pick].contiguous()
    sh = (torch.from_numpy(rows).to(dev()), torch.from_numpy(ids).to(dev())[pick].contiguous()) if shift else (None, None)
    want = torch.from_numpy(want).to(dev())[pick]
    assert torch.equal(qb.pq_encode(idx, xs, *sh), want)
    flat = torch.empty(xs.numel() + 1, device=dev())  # an address that allows no wide loads
    flat[1:] = xs.view(-1)
    assert torch.equal(qb.pq_encode(idx, flat[1:].view(n, d), *sh), want)
    idx.close()


@pytest.mark.parametrize("d,m", [(64, 16), (96, 16), (128, 16), (96, 32), (128, 32)])
@pytest.mark.parametrize("kind", ["skewed", "integer", "unbounded", "largest"])
def test_encode_matrix_form(qb, d, m, kind):
    """The products on the matrix cores: counts around a wave's tile of 16 vectors and around its second tile
    (3072 waves), sub-spaces of very different size (what decides is small beside the vector's norm), many equal
    distances, vectors with infinities and NaN in one sub-space, which must not touch the others, and norms around
    the largest that the expanded form may take (sums of products overflow above them)."""
    lay = synth.make_layout(d, [4] * m, 16)
    rng = np.random.default_rng(d + m)
    ds = d // m
    cb = rng.normal(size=(m, 16, ds)).astype(np.float32)
    x = rng.normal(size=(700, m, ds)).astype(np.float32)
    if kind == "skewed":
        s = np.float32(10.0) ** rng.integers(-9, 10, (m, 1))
        cb, x = cb * s[:, None, :], x * s[None]
    elif kind == "integer":
        cb, x = np.round(2 * cb), np.round(2 * x)
    elif kind == "largest":
        s = np.float32(10.0) ** rng.uniform(18.0, 19.3, (m, 1))
        cb, x = cb * s[:, None, :], x * s[None]
    else:
        x[::3, 1, 0] = np.inf
        x[1::3, m - 1, ds - 1] = -np.inf
        cb[2, 5] = 3e38
    cb, x = cb.astype(np.float32).reshape(-1), x.astype(np.float32).reshape(700, d)
    with np.errstate(all="ignore"):
        want = torch.from_numpy(oracle.encode(d, lay.nbits, lay.dsub, cb, x)).to(dev())
    idx = qb.PqIndex(lay.d, lay.nbits, lay.dsub, torch.from_numpy(cb).to(dev()), 8)
    for n in (1, 15, 16, 17, 63, 64, 65, 3072 * 16 + 1, 3 * 3072 * 16 - 5):
        pick = torch.arange(n, device=dev()) % 700
        assert torch.equal(qb.pq_encode(idx, torch.from_numpy(x).to(dev())[pick].contiguous()), want[pick]), n
    idx.close()


@pytest.mark.parametrize("d,m", [(96, 16), (128, 32), (100, 5)])
@pytest.mark.parametrize("n", [64 * 0x7FFFFFFF + 1, 1 << 62, (1 << 63) - 1])
def test_encode_refuses_more_vectors_than_a_call_can_take(qb, d, m, n):
    """Every form refuses the same n (before anything is launched)."""
    lay = synth.make_layout(d, [4] * m, 16)
    cb = torch.zeros(sum(16 * s for s in lay.dsub), device=dev())
    idx = qb.PqIndex(lay.d, lay.nbits, lay.dsub, cb, 8)
    x, codes = torch.zeros((64, d), device=dev()), torch.zeros((64, 16), dtype=torch.uint8, device=dev())
    assert qb.load().pq_encode(idx.handle, x.data_ptr(), n, None, None, codes.data_ptr(), None) == qb.PQ_EINVAL
    assert b"too large" in qb.load().pq_last_error()
    idx.close()


@pytest.mark.parametrize("d,m", [(96, 16), (128, 32)])
def test_encode_matrix_form_decides_uneven_sub_spaces_itself(qb, d, m):
    """Near ties are told by the sub-space's own size: vectors whose first dimensions, or one sub-space, carry nearly all
    of the norm take about as long as even ones.  (With the whole vector's norm every other sub-space counted as a near tie
    and was encoded twice: 1.5 to 2 times as long.)"""
    lay = synth.make_layout(d, [4] * m, 16)
    ds, g = d // m, torch.Generator(device=dev()).manual_seed(5)
    scales = {"even": torch.ones(d), "falling": 1.0 / torch.arange(1.0, d + 1.0) ** 2, "one large": torch.ones(d)}
    scales["one large"][ds:2 * ds] = 1000.0
    calls = {}
    for name, sc in scales.items():
        x = torch.randn((500_000, d), generator=g, device=dev()) * sc.to(dev())
        cb = x[:16].view(16, m, ds).transpose(0, 1).contiguous().view(-1)
        calls[name] = (qb.PqIndex(lay.d, lay.nbits, lay.dsub, cb, 8), x, [])
    for rep in range(12):
        for idx, x, t in calls.values():
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(10):
                qb.pq_encode(idx, x)
            b.record()
            b.synchronize()
            t.append(a.elapsed_time(b))
    med = {name: sorted(t)[6] for name, (_, _, t) in calls.items()}
    for idx, _, _ in calls.values():
        idx.close()
    assert max(med.values()) < 1.35 * med["even"], med
