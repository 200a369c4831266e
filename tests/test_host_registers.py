"""What the compiler made of the kernels, from the code objects inside libhgnn.so: loops that spill registers read and write memory for it in every round."""
import re
import struct

import pytest

from paper_2411_01109_amd import build as hip_build

msgpack = pytest.importorskip("msgpack")


def kernels():
    """-> {kernel: what its code object says of it} of the library"""
    with open(hip_build.LIB_PATH, "rb") as fh:
        lib = fh.read()
    out, at = {}, lib.find(b"\x7fELF", 1)
    while at >= 0:
        if lib[at + 4:at + 6] == b"\x02\x01" and struct.unpack_from("<H", lib, at + 18)[0] == 224:  # AMDGPU
            shoff = struct.unpack_from("<Q", lib, at + 40)[0]
            size, n = struct.unpack_from("<HH", lib, at + 58)
            for i in range(n):
                kind, _, _, offset, length = struct.unpack_from("<IQQQQ", lib, at + shoff + i * size + 4)
                if kind != 7:  # SHT_NOTE
                    continue
                p, end = at + offset, at + offset + length
                while p < end:
                    namesz, descsz, what = struct.unpack_from("<III", lib, p)
                    desc = p + 12 + (namesz + 3) // 4 * 4
                    if what == 32:
                        out.update((k[".name"], k) for k in msgpack.unpackb(lib[desc:desc + descsz])["amdhsa.kernels"])
                    p = desc + (descsz + 3) // 4 * 4
        at = lib.find(b"\x7fELF", at + 4)
    return out


def test_backward_of_attention_spills_nothing(hgnn):
    """The pass over the transposed graph (the third argument, VEC, is true)."""
    ours = {n: k for n, k in kernels().items() if re.search(r"gat_bwd_task_kernelILi\d+ELb[01]ELb1E", n)}
    assert len(ours) > 20
    spilled = {n: k[".private_segment_fixed_size"] for n, k in ours.items() if k[".private_segment_fixed_size"] or k[".vgpr_spill_count"]}
    assert not spilled


def test_dot_products_of_short_rows_keep_to_five_waves(hgnn):
    """Rows of 32 bytes: a SIMD's 512 registers hold five waves of 81 to 96."""
    ours = {n: k[".vgpr_count"] for n, k in kernels().items() if "sddmm_task_kernelILi2ELb1ELb0ELi2ELi8E" in n}
    assert ours and all(80 < v <= 96 for v in ours.values()), ours
