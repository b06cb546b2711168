"""Register spills of the built kernels, from the metadata of the library's own code
objects: the inner loops of the prefill are register-bound, and a kernel that spills
there loses more than any of its other costs."""
import struct

import msgpack
import pytest

from paper_2609_33135_amd import build

MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _kernels(path):
    """{name: metadata} over the AMDGPU code objects bundled in a shared library."""
    data, out = open(path, "rb").read(), {}
    at = data.find(MAGIC)
    while at >= 0:
        entry = at + len(MAGIC) + 8
        for _ in range(struct.unpack_from("<Q", data, at + len(MAGIC))[0]):
            off, size, n = struct.unpack_from("<QQQ", data, entry)
            target = data[entry + 24:entry + 24 + n]
            entry += 24 + n
            if b"gfx" in target and size:
                out.update(_notes(data[at + off:at + off + size]))
        at = data.find(MAGIC, at + 1)
    return out


def _notes(elf):
    table, = struct.unpack_from("<Q", elf, 40)
    width, count = struct.unpack_from("<HH", elf, 58)
    for i in range(count):
        if struct.unpack_from("<I", elf, table + i * width + 4)[0] == 7:   # SHT_NOTE
            at, _ = struct.unpack_from("<QQ", elf, table + i * width + 24)
            name, desc = struct.unpack_from("<II", elf, at)
            at += 12 + (name + 3) // 4 * 4
            return {k[".name"]: k for k in msgpack.unpackb(elf[at:at + desc])["amdhsa.kernels"]}
    return {}


@pytest.fixture(scope="module")
def kernels():
    import paper_2609_33135_amd as mp
    mp.lib()
    return _kernels(build.LIB)


# prefill_kernel<SEED, MX, PV, ABL>: NVFP4 PV (2), without and with the compensation (accumulator input)
@pytest.mark.parametrize("seed", [0, 2])
def test_nvfp4_pv_prefill_does_not_spill(kernels, seed):
    found = [k for n, k in kernels.items() if f"prefill_kernelILi{seed}ELb0ELi2ELi0E" in n]
    assert len(found) == 1, sorted(kernels)
    assert found[0][".vgpr_spill_count"] == 0 and found[0][".private_segment_fixed_size"] == 0
