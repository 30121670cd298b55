"""Registers of the reverse kernels, read from the metadata of the code objects
in the built library: FP64 reverse steps hold psi_0's gradient, the running
sums and the node's values in 256 registers, and what does not fit goes through
scratch memory, which bounded them once (584 bytes a lane at two sweeps, where
loads a transform ahead of their use took 80 registers: 30 % of a reverse step
with the chip full).  The bounds are the largest of the kernels that load where
they use, 320 and 536 bytes a lane at two and three sweeps."""
import re
import struct

import msgpack
import pytest

from paper_1101_0086_amd import _lib

MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _code_objects(blob):
    at = blob.find(MAGIC)
    while at >= 0:
        (count,) = struct.unpack_from("<Q", blob, at + len(MAGIC))
        p = at + len(MAGIC) + 8
        for _ in range(count):
            off, size, n = struct.unpack_from("<QQQ", blob, p)
            triple = blob[p + 24:p + 24 + n]
            p += 24 + n
            if b"gfx950" in triple and size:
                yield blob[at + off:at + off + size]
        at = blob.find(MAGIC, p)


def _kernels(elf):
    """Kernel metadata (name -> dict) of an ELF's AMDGPU note (type 32, msgpack)."""
    shoff, = struct.unpack_from("<Q", elf, 0x28)
    entsize, num = struct.unpack_from("<HH", elf, 0x3A)
    out = {}
    for i in range(num):
        kind, = struct.unpack_from("<I", elf, shoff + i * entsize + 4)
        off, size = struct.unpack_from("<QQ", elf, shoff + i * entsize + 0x18)
        if kind != 7:                                   # SHT_NOTE
            continue
        p = off
        while p < off + size:
            nlen, dlen, ntype = struct.unpack_from("<III", elf, p)
            d = p + 12 + (nlen + 3) // 4 * 4
            if ntype == 32 and elf[p + 12:p + 12 + nlen].startswith(b"AMDGPU"):
                for k in msgpack.unpackb(elf[d:d + dlen])["amdhsa.kernels"]:
                    out[k[".name"]] = k
            p = d + (dlen + 3) // 4 * 4
    return out


@pytest.fixture(scope="module")
def kernels():
    with open(_lib.LIB_PATH, "rb") as f:
        blob = f.read()
    out = {}
    for elf in _code_objects(blob):
        out.update(_kernels(elf))
    return out


@pytest.mark.parametrize("nit,bound", [(2, 320), (3, 536)])
def test_fp64_reverse_kernels_fit(kernels, nit, bound):
    got = {}
    for name, k in kernels.items():
        m = re.search(r"mpa_adjoint_block_kernelIdLi(\d+)ELi(\d+)ELi(\d+)E", name)
        if m and int(m.group(2)) == nit:
            got[int(m.group(1)), int(m.group(3))] = k[".private_segment_fixed_size"]
    assert {b for b, _ in got} == {512, 1024, 2048, 4096}
    assert max(got.values()) <= bound, got
