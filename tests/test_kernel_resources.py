"""Host-only: the built library's kernels keep their values in registers.  What
spills costs a round trip to scratch memory per use, and nothing else shows it."""

import os
import struct

import msgpack
import pytest

from paper_2608_03893_amd import build

# Scratch bytes per lane that a kernel may use: topk's list for NaN scores, which a
# variable indexes; elsewhere a few values at the kernel's register limit.
ALLOWED = {"topk_kernel": 272, "gram_kernel": 12, "xhead_gemm_kernel": 12, "mlp_gemm_kernelILi3": 36,
           "map_w_kernelILi3": 28, "map_w_kernelILi4": 12}


def kernels():
    """(name, scratch bytes per lane, spilled VGPRs) of every kernel in the
    library, from the metadata notes of its code objects."""
    data = open(build.LIB, "rb").read()
    out, at = [], data.find(b"\x7fELF", 1)
    while at >= 0:
        if data[at + 18:at + 20] == struct.pack("<H", 224):   # EM_AMDGPU
            phoff, = struct.unpack_from("<Q", data, at + 32)
            phsize, phnum = struct.unpack_from("<HH", data, at + 54)
            for n in range(phnum):
                kind, _, off, _, _, size = struct.unpack_from("<IIQQQQ", data, at + phoff + n * phsize)
                p, end = at + off, at + off + size
                while kind == 4 and p < end:                   # PT_NOTE
                    namesz, descsz, ntype = struct.unpack_from("<III", data, p)
                    desc = p + 12 + (namesz + 3) // 4 * 4
                    if ntype == 32 and data[p + 12:p + 18] == b"AMDGPU":
                        for k in msgpack.unpackb(data[desc:desc + descsz])["amdhsa.kernels"]:
                            out.append((k[".name"], k[".private_segment_fixed_size"], k[".vgpr_spill_count"]))
                    p = desc + (descsz + 3) // 4 * 4
        at = data.find(b"\x7fELF", at + 4)
    return out


@pytest.fixture(scope="module")
def built():
    if not os.path.exists(build.LIB):
        build.build()
    return kernels()


def test_kernels_do_not_spill(built):
    assert any("fit_solve_kernel" in n for n, _, _ in built)
    for name, scratch, spilled in built:
        most = next((b for s, b in ALLOWED.items() if s in name), 0)
        assert scratch <= most, f"{name}: {scratch} bytes of scratch, {spilled} registers spilled"
