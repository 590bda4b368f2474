"""The half-precision form of the coarse search (batches over many cells) must return, byte for byte,
what the exact matrix form returns, on data of any scale, with ties, and where its bound fails and the
exact form has to take over."""
import numpy as np
import pytest
import torch

import oracle
from harness import synth
from paper_1812_09162_amd import binding as qb

pytestmark = pytest.mark.gpu


def _data(kind, n, d, seed):
    x = synth.GENERATORS["gamma_ints" if kind == "gamma" else "aniso_gauss"](n, d, seed)
    if kind == "offset":      # all vectors close together, far from the origin
        x = x + 30.0
    elif kind == "tiny":
        x = x * 1e-9
    elif kind == "huge":
        x = x * 1e9
    elif kind == "ties":      # small integers: many equal scores
        x = torch.round(x * 8.0)
    elif kind == "spread":    # components of very different size
        x = x * torch.logspace(-6, 3, d)
    return x.cuda()


def _matrix(z, c, nprobe):
    qb.pq_set_option(qb.PQ_OPT_COARSE_FILTER, 0)
    try:
        return qb.ivf_coarse_search(z, c, nprobe)
    finally:
        qb.pq_set_option(qb.PQ_OPT_COARSE_FILTER, 1)


def _same(got, want):
    assert torch.equal(got[0], want[0])
    assert torch.equal(got[1].view(torch.int32), want[1].view(torch.int32))


def _check(z, c, nprobe, half=False):
    if half:
        assert qb.ivf_coarse_form(z.shape[0], c.shape[0], c.shape[1], nprobe) == qb.PQ_COARSE_HALF
    _same(qb.ivf_coarse_search(z, c, nprobe), _matrix(z, c, nprobe))


@pytest.mark.parametrize("kind", ["gauss", "gamma", "offset", "tiny", "huge", "ties", "spread"])
@pytest.mark.parametrize("nq,K,d,nprobe", [(64, 16384, 96, 64), (131, 20_011, 128, 33), (97, 33_001, 109, 1)])
def test_kinds_of_data(kind, nq, K, d, nprobe):
    _check(_data(kind, nq, d, 5), _data(kind, K, d, 6), nprobe)


@pytest.mark.parametrize("zs,cs", [(1e-21, 1e-21), (3e-22, 3e-22), (1e-22, 1e-22), (1e-20, 1e-22), (3e-18, 3e-18),
                                   (3e20, 3e18), (1e20, 1e17), (1e15, 1e15)])
def test_products_outside_the_normal_range(zs, cs):
    """Products that underflow leave the definition's chain with few distinct scores (ties: the lowest ids);
    products that overflow leave scores of -inf."""
    z, c = _data("gauss", 70, 96, 21) * zs, _data("gauss", 20_000, 96, 22) * cs
    _check(z, c, 20, half=True)
    ids, scores = qb.ivf_coarse_search(z, c, 20)
    for q in (0, 69):
        oi, osc = oracle.coarse_search(c.cpu().numpy(), z[q].cpu().numpy(), 20)
        assert np.array_equal(ids[q].cpu().numpy(), oi) and np.array_equal(scores[q].cpu().numpy(), osc)


@pytest.mark.parametrize("d", [1, 13, 110, 125, 126, 142, 200, 256, 257])
def test_dimensions(d):
    _check(_data("gauss", 70, d, 7), _data("gauss", 17_000, d, 8), 40)


@pytest.mark.parametrize("nq,K,nprobe", [(4100, 65_536, 64), (600, 65_543, 256), (64, 131_072, 200)])
def test_sizes(nq, K, nprobe):
    _check(_data("gauss", nq, 96, 9), _data("gauss", K, 96, 10), nprobe)


@pytest.mark.parametrize("kind", ["gauss", "gamma", "offset", "tiny", "huge", "ties", "spread"])
@pytest.mark.parametrize("nq,K,d,nprobe", [(64, 16_384, 96, 20), (128, 20_011, 128, 21), (97, 32_768, 109, 1), (300, 70_001, 100, 80)])
def test_kinds_of_data_in_half_precision(kind, nq, K, d, nprobe):
    _check(_data(kind, nq, d, 5), _data(kind, K, d, 6), nprobe, half=True)


@pytest.mark.parametrize("d,nq", [(16, 1000), (33, 1000), (48, 257), (96, 300), (108, 70), (109, 300), (110, 70), (125, 300),
                                  (126, 70), (140, 300), (141, 300), (142, 300), (200, 70), (252, 300), (253, 70), (256, 300)])
def test_dimensions_in_half_precision(d, nq):
    """edges of the 7, 9 and 18 steps of 16 columns"""
    _check(_data("gauss", nq, d, 7), _data("gauss", 17_000, d, 8), 20, half=True)


@pytest.mark.parametrize("nq,K,nprobe", [(600, 65_543, 80), (300, 262_144, 300), (129, 131_072, 160), (200, 1_000_003, 60), (4097, 65_600, 1), (257, 16_384, 1)])
def test_sizes_in_half_precision(nq, K, nprobe):
    _check(_data("gauss", nq, 96, 9), _data("gauss", K, 96, 10), nprobe, half=True)


def test_where_the_lists_or_the_range_do_not_suffice_in_half_precision():
    """calls that the exact form has to take over, in whole or for one of several passes"""
    z, c = _data("gauss", 80, 96, 11), _data("gauss", 20_000, 96, 12)
    order = (c - z[0]).square().sum(1).argsort()
    _check(z, c[order].contiguous(), 20, half=True)                      # the nearest cells of a query side by side
    _check(z, c[order.flip(0)].contiguous(), 20, half=True)
    _check(z, c[:50].repeat(400, 1).contiguous(), 20, half=True)         # every cell 400 times: more than a block picks from
    _check(torch.cat([z[:70], z[70:] * 1e6]), c, 20, half=True)          # queries beyond the cells' range
    _check(z * 0.0, c, 20, half=True)
    _check(z, c * 0.0, 20, half=True)
    few = c.clone()
    few[1000:] = c[1000:1001]                                            # one cell 19,000 times, far from or near to a query
    _check(z, few, 20, half=True)
    _check(torch.cat([z[:70], few[1000:1001].repeat(10, 1)]), few, 20, half=True)


def test_where_the_lists_or_the_range_do_not_suffice():
    z, c = _data("gauss", 80, 96, 11), _data("gauss", 20_000, 96, 12)
    order = (c - z[0]).square().sum(1).argsort()
    _check(z, c[order].contiguous(), 64)                      # the nearest cells of a query side by side
    _check(z, c[:50].repeat(400, 1).contiguous(), 64)         # every cell 400 times
    _check(torch.cat([z[:70], z[70:] * 1e6]), c, 64)          # queries beyond the cells' range
    _check(z * 0.0, c, 64)
    _check(z, c * 0.0, 64)


@pytest.mark.parametrize("nq,K,d", [(64, 65_536, 250), (300, 16_384, 96), (5000, 65_600, 40)])
def test_smallest_workspace(nq, K, d):
    """with no more workspace than the matrix form needs: the half-precision form where it fits, else another;
    several passes, one of which the exact form takes over"""
    z, c = _data("gauss", nq, d, 23), _data("gauss", K, d, 24)
    z[nq // 2] *= 1e7
    least = qb.ivf_coarse_workspace_bytes(nq, K)
    while True:
        try:
            qb.ivf_coarse_form(nq, K, d, 20, least - 256)
        except qb.QadcError:
            break
        least -= 256
    got = qb.ivf_coarse_search(z, c, 20, workspace=torch.empty(least, dtype=torch.uint8, device="cuda"))
    _same(got, _matrix(z, c, 20))
    _check(z, c, 20)


@pytest.mark.parametrize("kind", ["gauss", "gamma", "ties"])
@pytest.mark.parametrize("nq,K,d,nprobe", [(1, 65_536, 96, 64), (2, 63, 20, 5), (4, 8192, 33, 64), (5, 8191, 32, 64),
                                           (16, 70_001, 128, 1), (16, 300, 97, 300), (9, 300_000, 16, 1024), (3, 40_000, 1, 7)])
def test_few_queries(kind, nq, K, d, nprobe):
    """calls of up to 16 queries take the direct form: as rows of a larger batch in the matrix form"""
    z, c = _data(kind, 20, d, 13), _data(kind, K, d, 14)
    qb.pq_set_option(qb.PQ_OPT_COARSE_FILTER, 0)
    try:
        want = qb.ivf_coarse_search(z, c, nprobe)
    finally:
        qb.pq_set_option(qb.PQ_OPT_COARSE_FILTER, 1)
    got = qb.ivf_coarse_search(z[:nq].contiguous(), c, nprobe)
    assert torch.equal(got[0], want[0][:nq])
    assert torch.equal(got[1].view(torch.int32), want[1][:nq].view(torch.int32))
