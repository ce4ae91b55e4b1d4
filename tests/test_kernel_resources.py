"""Scratch memory (spilled registers) of the built regression kernels, from the
code objects' metadata in libesim.so: instances whose sums do not stay in registers
run several times slower (a window's every row then goes through scratch)."""
import os
import re
import struct

import msgpack
import pytest

from paper_2303_02608_amd import binding as B


def _kernels(path):
    """Metadata of every gfx950 kernel in the library: symbol -> record."""
    data = open(path, "rb").read()
    out = {}
    at = data.find(b"\x7fELF", 4)
    while at >= 0:
        if struct.unpack_from("<H", data, at + 18)[0] == 224:        # EM_AMDGPU
            phoff, = struct.unpack_from("<Q", data, at + 32)
            phsize, phnum = struct.unpack_from("<HH", data, at + 54)
            for i in range(phnum):
                kind, _, off, _, _, size = struct.unpack_from("<IIQQQQ", data, at + phoff + i * phsize)
                p, end = at + off, at + off + size
                while kind == 4 and p + 12 <= end:                   # PT_NOTE
                    nlen, dlen, ntype = struct.unpack_from("<III", data, p)
                    desc = p + 12 + (nlen + 3) // 4 * 4
                    if ntype == 32 and data[p + 12:p + 12 + nlen].rstrip(b"\0") == b"AMDGPU":
                        meta = msgpack.unpackb(data[desc:desc + dlen], strict_map_key=False)
                        out.update((k[".name"], k) for k in meta["amdhsa.kernels"])
                    p = desc + (dlen + 3) // 4 * 4
        at = data.find(b"\x7fELF", at + 4)
    return out


@pytest.fixture(scope="module")
def kernels():
    if not os.path.exists(B.LIB_PATH):
        pytest.skip("libesim.so is not built")
    k = _kernels(B.LIB_PATH)
    assert len(k) > 100
    return k


def _scratch(kernels, pattern):
    """Scratch bytes per lane of the kernels whose mangled name holds pattern."""
    got = [k[".private_segment_fixed_size"] for n, k in kernels.items() if re.search(pattern, n)]
    assert got, pattern
    return max(got)


# regress_kernel<F, L, f16, c32, kappa>, bandwidth_dense_kernel<F, f16>; the bytes before these kernels
# kept one walk's sums over the branches of all frame counts (F = 12 half precision: 980)
@pytest.mark.parametrize("F,lanes,dense,kappa", [(7, 208, 180, 830), (8, 416, 330, 1356), (10, 16, 64, 1460),
                                                 (12, 980, 980, 2412)])
def test_windows_from_memory(kernels, F, lanes, dense, kappa):
    for L in (1, 2):
        assert _scratch(kernels, rf"regress_kernelILi{F}ELi{L}ELb[01]ELb0ELb0E") <= lanes
    assert _scratch(kernels, rf"bandwidth_dense_kernelILi{F}E") <= dense
    assert _scratch(kernels, rf"regress_kernelILi{F}ELi1ELb[01]ELb0ELb1E") <= kappa


@pytest.mark.parametrize("F", [1, 3, 5, 7])
def test_tiles_and_default_lists_stay_in_registers(kernels, F):
    assert _scratch(kernels, rf"regress_tile_kernelILi{F}E") == 0
    for kind in (0, 1):
        assert _scratch(kernels, rf"regress_list_kernelILi{F}ELi16ELb[01]ELi{kind}E") <= 48


# (with an item's fields and best SURE held over the walks: 160 and 308 bytes)
@pytest.mark.parametrize("F,limit", [(7, 80), (8, 240)])
def test_bandwidth_lists(kernels, F, limit):
    assert _scratch(kernels, rf"bandwidth_list_kernelILi{F}ELb[01]ELi1E") <= limit
