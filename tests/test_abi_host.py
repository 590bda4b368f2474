"""CPU-side checks of the C-ABI library: it loads, exports every function that
include/qadc.h declares, and rejects bad arguments with an error code and a message
(no compute call is made here: there is no GPU in this tier)."""
import ctypes
import os
import re

import pytest

from paper_1812_09162_amd import binding as qb

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def declared_functions():
    text = "".join(open(os.path.join(ROOT, "include", h)).read() for h in ("qadc.h", "qadc_bench.h"))
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b((?:pq|ivf)_[a-z_]+)\s*\(", text)))


def test_library_exports_every_declared_symbol():
    lib = qb.load()
    names = declared_functions()
    assert len(names) >= 13
    for n in names:
        assert hasattr(lib, n), n
    assert set(names) == set(qb.EXPORTS)


def test_qparams_record_is_24_bytes():
    import numpy as np
    rec = np.dtype([("d_min", "<f8"), ("delta", "<f8"), ("d_max", "<f4"), ("key_bound", "<u4")])
    assert rec.itemsize == qb.QPARAMS_BYTES


def test_index_create_rejects_bad_shapes_before_touching_the_gpu():
    lib = qb.load()
    h = ctypes.c_void_p()

    def create(d, nbits, dsub, acc, cb=0x1000):
        nb = (ctypes.c_int32 * len(nbits))(*nbits)
        ds = (ctypes.c_int32 * len(dsub))(*dsub)
        return lib.pq_index_create(ctypes.byref(h), d, len(nbits), ctypes.cast(nb, ctypes.c_void_p),
                                   ctypes.cast(ds, ctypes.c_void_p), cb, acc)

    assert create(8, [4, 4], [4, 4], 12) == qb.PQ_EINVAL          # acc_bits
    assert b"acc_bits" in lib.pq_last_error()
    assert create(8, [4, 9], [4, 4], 8) == qb.PQ_EINVAL           # nbits out of range
    assert create(8, [4, 4], [4, 3], 8) == qb.PQ_EINVAL           # sum(dsub) != d
    assert b"sum(dsub)" in lib.pq_last_error()
    assert create(8, [4, 4], [8, 0], 8) == qb.PQ_EINVAL           # empty sub-vector
    assert create(8, [4, 4], [4, 4], 8, cb=None) == qb.PQ_EINVAL  # null codebooks
    assert create(0, [4], [0], 8) == qb.PQ_EINVAL
    assert create(17 * 8, [8] * 17, [8] * 17, 8) == qb.PQ_EINVAL  # table longer than the limit
    assert h.value is None


def test_options_are_validated_and_kept():
    lib = qb.load()
    assert lib.pq_get_option(qb.PQ_OPT_SCAN_BLOCKS) == 2048
    assert lib.pq_set_option(qb.PQ_OPT_SCAN_BLOCKS, 0) == qb.PQ_EINVAL       # out of range: unchanged
    assert lib.pq_set_option(qb.PQ_OPT_IVF_THREADS, 100) == qb.PQ_EINVAL
    assert lib.pq_set_option(qb.PQ_OPT_IVF_SHARED_LISTS, 3) == qb.PQ_EINVAL
    assert lib.pq_get_option(qb.PQ_OPT_IVF_SHARED_LISTS) == 1
    assert lib.pq_set_option(99, 1) == qb.PQ_EINVAL and b"option 99" in lib.pq_last_error()
    assert lib.pq_get_option(99) == -1
    assert lib.pq_set_option(qb.PQ_OPT_SCAN_BLOCKS, 1024) == qb.PQ_OK
    assert lib.pq_get_option(qb.PQ_OPT_SCAN_BLOCKS) == 1024
    assert lib.pq_set_option(qb.PQ_OPT_SCAN_BLOCKS, 2048) == qb.PQ_OK


def test_calls_reject_null_handle():
    lib = qb.load()
    assert lib.pq_compute_tables(None, None, 1, None, None) == qb.PQ_EINVAL
    assert lib.pq_quantize_tables(None, None, 1, None, 0, 400, 10, None, None, None) == qb.PQ_EINVAL
    assert lib.pq_adc_scan_topk(None, None, None, 1, None, 0, 10, None, None, None, None, 0,
                                None) == qb.PQ_EINVAL
    assert lib.ivf_adc_scan_topk(None, None, 1, None, None, None, None, 1, None, 1, 400, 10, None,
                                 None, None, 0, None) == qb.PQ_EINVAL
    assert lib.ivf_adc_scan_topk_tightening(None, None, 1, None, None, None, None, 1, None, 1, 400, 10,
                                            None, None, None, 0, None) == qb.PQ_EINVAL
    assert b"ivf_adc_scan_topk_tightening" in lib.pq_last_error()
    assert lib.pq_code_size(None) == 0 and lib.pq_table_len(None) == 0
    assert lib.pq_workspace_bytes(None, 1, 10, 10) == 0
    lib.pq_index_destroy(None)


def _coarse_bytes_without_half_form(nq, K):
    """norms, score matrix, and the candidate lists of the filtering form (32 entries per 256 cells)"""
    def up(x):
        return (x + 255) // 256 * 256
    ld, ncb = (K + 31) // 32 * 32, (K + 255) // 256
    qc = min(max((1 << 30) // (4 * ld) // 128 * 128, 128), (nq + 127) // 128 * 128)
    return up(4 * K) + up(qc * ld * 4) + up(qc * ncb * 256) + up(qc * ncb * 4) + 2 * up(qc * 1024 * 4) + 256


@pytest.mark.parametrize("nq,K", [(1, 100), (16, 65_536), (63, 65_536), (64, 16_384), (100, 20_011), (128, 65_536),
                                  (1000, 65_536), (4097, 65_536), (10_000, 65_536), (256, 1 << 20), (1000, 1_000_000)])
def test_coarse_workspace_keeps_within_what_the_matrix_form_needs(nq, K):
    """A workspace of the matrix form's size is accepted, whichever form would run with more; the size asked
    for is hardly larger (the matrix has room for the half-precision form's lists)."""
    least, asked = _coarse_bytes_without_half_form(nq, K), qb.ivf_coarse_workspace_bytes(nq, K)
    assert least <= asked <= 1.4 * least
    for d, nprobe in ((96, 64), (256, 1), (257, 1024)):
        assert qb.ivf_coarse_form(nq, K, d, nprobe, least) in (qb.PQ_COARSE_MATRIX, qb.PQ_COARSE_FILTER,
                                                               qb.PQ_COARSE_HALF, qb.PQ_COARSE_DIRECT)
        with pytest.raises(qb.QadcError) as e:
            qb.ivf_coarse_form(nq, K, d, nprobe, least - 1)
        assert e.value.code == qb.PQ_ENOMEM
    # 96 and 128 dimensions over 65,536 cells, long batches: also with the smaller workspace
    if nq >= 1000 and K == 65_536:
        assert least == asked
    for nq2 in (129, 1000, 10_000):
        assert qb.ivf_coarse_form(nq2, 65_536, 96, 64, _coarse_bytes_without_half_form(nq2, 65_536)) == qb.PQ_COARSE_HALF


def test_which_coarse_form():
    """The lines between the forms: nq, K, d, nprobe."""
    H, F, M, D = qb.PQ_COARSE_HALF, qb.PQ_COARSE_FILTER, qb.PQ_COARSE_MATRIX, qb.PQ_COARSE_DIRECT
    for call, form in (((1, 65_536, 96, 64), D), ((16, 300, 97, 300), D), ((17, 65_536, 96, 64), F), ((63, 16_384, 96, 20), F),
                       ((64, 16_384, 96, 20), H), ((64, 16_384, 96, 22), F), ((128, 32_768, 96, 32), H), ((128, 32_769, 96, 32), F),
                       ((129, 65_536, 96, 64), H), ((200, 65_536, 64, 64), F), ((256, 65_536, 144, 64), F), ((257, 65_536, 144, 64), H),
                       ((257, 65_536, 64, 64), H), ((999, 65_536, 32, 64), F), ((1000, 65_536, 32, 64), H), ((1000, 200_000, 32, 64), F),
                       ((1000, 65_536, 15, 64), F), ((1000, 1_000_000, 96, 64), H), ((1000, 1_000_000, 96, 84), F), ((1000, 262_144, 96, 300), H),
                       ((1000, 16_384, 96, 64), F), ((1000, 16_000, 96, 1), M), ((1000, 65_536, 257, 64), F), ((1000, 300, 96, 64), M)):
        assert qb.ivf_coarse_form(*call) == form, call
