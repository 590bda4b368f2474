"""Registers of the kernels whose speed hangs on how many wavefronts a SIMD holds (512 registers a lane, handed out in
eights), as the compiler reports them in the built library's own metadata."""
import struct

import msgpack
import pytest

from paper_1812_09162_amd.binding import LIB_PATH


def kernels():
    """name -> (registers, bytes of scratch memory) of every kernel in the library's gfx950 code objects"""
    blob, out, at = open(LIB_PATH, "rb").read(), {}, 0
    while (at := blob.find(b"\x7fELF\x02", at + 1)) > 0:
        if struct.unpack_from("<H", blob, at + 18)[0] != 224:  # EM_AMDGPU
            continue
        shoff, = struct.unpack_from("<Q", blob, at + 40)
        entsize, count = struct.unpack_from("<HH", blob, at + 58)
        for i in range(count):
            kind, = struct.unpack_from("<I", blob, at + shoff + i * entsize + 4)
            if kind != 7:  # SHT_NOTE
                continue
            off, size = struct.unpack_from("<QQ", blob, at + shoff + i * entsize + 24)
            nlen, dlen, ntype = struct.unpack_from("<III", blob, at + off)
            assert ntype == 32 and 12 + nlen + dlen <= size + 8  # NT_AMDGPU_METADATA
            for k in msgpack.unpackb(blob[at + off + 12 + (nlen + 3) // 4 * 4:][:dlen])["amdhsa.kernels"]:
                out[k[".name"]] = (k[".vgpr_count"], k[".private_segment_fixed_size"])
    return out


@pytest.mark.parametrize("name,waves", [
    ("k_scan_mxILi5ELi18ELi1ELi801E", 2),  # {6,6,4} x 8, one query tile: one wave exposes the reads of its rows
    ("k_scan_mxILi5ELi16ELi1ELi440E", 2),
    ("k_scan_mxILi1ELi4ELi1ELi0E", 5),     # 16 x 4 bits, one to four query tiles
    ("k_scan_mxILi1ELi4ELi2ELi0E", 4),
    ("k_scan_mxILi1ELi4ELi3ELi0E", 3),
    ("k_scan_mxILi1ELi4ELi4ELi0E", 2),
    ("k_ivf_scan_mxILi6E", 7),
    ("k_ivf_scanILi1EhLi2ELi6E", 8),       # the inverted-list scan: the fixed shape, 8- and 16-byte codes
    ("k_ivf_scanILi1EhLi2ELi0E", 8),
    ("k_ivf_scanILi2EhLi4ELi0E", 8),
    ("k_ivf_scanILi3EtLi4ELi0E", 8),
    ("k_ivf_scanILi4EtLi2ELi0E", 8),
    ("k_ivf_scanILi5EtLi4ELi0E", 6),
    ("k_ivf_scanILi5EtLi0ELi0E", 6),
    *((f"k_ivf_tight_fixILi{ds}ELi{nr}E", 8) for ds in (4, 6, 8) for nr in (2, 4)),
    ("k_encode_mxILi16ELi6E", 3),
    ("k_quantizeILi1EhLi256E", 7),
    ("k_quantizeILi1EtLi256E", 7),
])
def test_wavefronts_a_simd_holds(name, waves):
    found = [v for k, v in kernels().items() if name in k]
    assert len(found) == 1
    regs, scratch = found[0]
    assert 512 // ((regs + 7) // 8 * 8) >= waves and scratch == 0, (regs, scratch)
