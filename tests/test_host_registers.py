"""What the compiler made of the kernels, from the code objects inside libhgnn.so: loops that spill registers read and write memory for it in every round."""
import re
import struct

import pytest

from paper_2411_01109_amd import build as hip_build

msgpack = pytest.importorskip("msgpack")


def kernels():
    """-> {kernel: what its code object says of it} of the library; "registers": what a wave is given of a SIMD's 512, in steps of eight"""
    with open(hip_build.LIB_PATH, "rb") as fh:
        lib = fh.read()
    out, at = {}, lib.find(b"\x7fELF", 1)
    while at >= 0:
        if lib[at + 4:at + 6] == b"\x02\x01" and struct.unpack_from("<H", lib, at + 18)[0] == 224:  # AMDGPU
            shoff = struct.unpack_from("<Q", lib, at + 40)[0]
            size, n = struct.unpack_from("<HH", lib, at + 58)
            sections = [struct.unpack_from("<IIQQQQII", lib, at + shoff + i * size) for i in range(n)]  # name, type, flags, address, offset, size, link, info
            ours, given = {}, {}
            for _, kind, _, _, offset, length, link, _ in sections:
                if kind == 7:  # SHT_NOTE
                    p, end = at + offset, at + offset + length
                    while p < end:
                        namesz, descsz, what = struct.unpack_from("<III", lib, p)
                        desc = p + 12 + (namesz + 3) // 4 * 4
                        if what == 32:
                            ours.update((k[".name"], k) for k in msgpack.unpackb(lib[desc:desc + descsz])["amdhsa.kernels"])
                        p = desc + (descsz + 3) // 4 * 4
                if kind == 11:  # SHT_DYNSYM: the kernels' descriptors, whose word at 48 begins with the registers
                    for p in range(at + offset, at + offset + length, 24):
                        name, _, _, index, value, _ = struct.unpack_from("<IBBHQQ", lib, p)
                        name = at + sections[link][4] + name
                        name = lib[name:lib.index(b"\0", name)].decode()
                        if name.endswith(".kd"):
                            where = at + value - sections[index][3] + sections[index][4]
                            given[name[:-3]] = 8 * ((struct.unpack_from("<I", lib, where + 48)[0] & 63) + 1)
            for name, k in ours.items():
                out[name] = dict(k, registers=given[name])
        at = lib.find(b"\x7fELF", at + 4)
    return out


def test_backward_of_attention_spills_nothing(hgnn):
    """The pass over the transposed graph (the third argument, VEC, is true)."""
    ours = {n: k for n, k in kernels().items() if re.search(r"gat_bwd_task_kernelILi\d+ELb[01]ELb1E", n)}
    assert len(ours) > 20
    spilled = {n: k[".private_segment_fixed_size"] for n, k in ours.items() if k[".private_segment_fixed_size"] or k[".vgpr_spill_count"]}
    assert not spilled


def test_dot_products_of_short_rows_keep_to_five_waves(hgnn):
    """Rows of 32 bytes: a SIMD's 512 registers hold five waves of 88 or 96."""
    ours = {n: k["registers"] for n, k in kernels().items() if "sddmm_task_kernelILi2ELb1ELb0ELi2ELi8E" in n}
    assert ours and all(v in (88, 96) for v in ours.values()), ours
