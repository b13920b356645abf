"""Registers, spills and code size of kernels that have been slower for more of them, read from the built library's own notes and symbols."""
import re
import struct

import pytest

from paper_2512_17970_amd import binding

msgpack = pytest.importorskip("msgpack")


def _kernels():
    """name -> (registers, spilled registers, code bytes) of every kernel in the library."""
    out = {}
    data = open(binding.lib_path(), "rb").read()
    for bundle in re.finditer(b"__CLANG_OFFLOAD_BUNDLE__", data):
        at, (count,) = bundle.end() + 8, struct.unpack_from("<Q", data, bundle.end())
        for _ in range(count):
            offset, size, length = struct.unpack_from("<QQQ", data, at)
            triple, at = data[at + 24:at + 24 + length], at + 24 + length
            if b"gfx950" not in triple:
                continue
            elf = data[bundle.start() + offset:bundle.start() + offset + size]
            sh, = struct.unpack_from("<Q", elf, 40)
            step, sections = struct.unpack_from("<HH", elf, 58)
            headers = [struct.unpack_from("<IIQQQQIIQQ", elf, sh + step * k) for k in range(sections)]
            sizes = {}
            for h in headers:
                if h[1] == 11:                                      # dynamic symbols
                    names = headers[h[6]][4]
                    for k in range(h[4], h[4] + h[5], 24):
                        name, info, _, _, _, bytes_ = struct.unpack_from("<IBBHQQ", elf, k)
                        if info & 15 == 2:
                            sizes[elf[names + name:elf.index(b"\0", names + name)].decode()] = bytes_
            for h in headers:
                if h[1] == 7:                                       # notes
                    length, described, kind = struct.unpack_from("<III", elf, h[4])
                    if kind == 32:
                        start = h[4] + 12 + (length + 3) // 4 * 4
                        for k in msgpack.unpackb(elf[start:start + described])["amdhsa.kernels"]:
                            out[k[".name"]] = (k[".vgpr_count"], k[".vgpr_spill_count"], sizes[k[".name"]])
    return out


@pytest.fixture(scope="module")
def kernels():
    return _kernels()


def _one(kernels, name, *args):
    mangled = f"{len(name)}{name}I" + "".join(f"Lb{int(a)}E" if isinstance(a, bool) else f"Li{a}E" for a in args) + "E"
    found = [v for k, v in kernels.items() if mangled in k]
    assert len(found) == 1, (mangled, len(kernels))
    return found[0]


@pytest.mark.parametrize("args,code", [((2, 16, 16, 1, 2, False, 2), 20000), ((2, 8, 16, 1, 2, False, 2), 19800), ((1, 8, 16, 1, 2, False, 2), 19900),
                                       ((2, 8, 16, 1, 2, True, 2), 20300), ((1, 4, 16, 1, 2, True, 2), 20500)])
def test_epilogue_of_the_batched_kernel(kernels, args, code):
    """14 + 2 wavefronts, bytes of code: 440 more, row addresses in the epilogue, cost up to 2 % of a call.  (The limits lie 150 above.)"""
    assert _one(kernels, "gemm_batch_kernel", *args)[2] <= code


# <M, V, SB, NT, RW, KW, D, GS, ONE> of gemm_centroid_kernel
@pytest.mark.parametrize("args,registers", [((1, 16, 4, 1, rw, 8 // rw, 4, 3, one), 128) for rw in (1, 2, 4) for one in (False, True)])
def test_two_workgroups_share_a_compute_unit(kernels, args, registers):
    """512 threads and a table of 64 KB: up to 128 registers leave room for a second workgroup, 130 do not."""
    assert _one(kernels, "gemm_centroid_kernel", *args)[0] <= registers


@pytest.mark.parametrize("args,spills", [((4, 16, 1, 1, 1, 8, 2, 0, False), 18), ((1, 8, 4, 4, 1, 8, 2, 4, False), 11), ((2, 4, 2, 2, 1, 8, 2, 3, False), 0),
                                         ((4, 8, 2, 2, 1, 8, 2, 3, False), 0), ((2, 4, 1, 1, 1, 8, 2, 3, False), 7)])
def test_spilled_registers(kernels, args, spills):
    """Instances that were up to 12 % slower with some more."""
    assert _one(kernels, "gemm_centroid_kernel", *args)[1] <= spills
