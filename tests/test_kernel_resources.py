"""Registers and scratch of the kernels in the built library, as the compiler recorded them in its code objects: what the
choice of tiles, and of waves a SIMD, rests on."""
import os
import re
import struct

import msgpack
import pytest

LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2511_21513_amd", "libintattn.so")
NT_AMDGPU_METADATA = 32


def notes(elf):
    """(type, descriptor) of the notes of a 64-bit little-endian ELF image."""
    shoff, = struct.unpack_from("<Q", elf, 0x28)
    shentsize, shnum = struct.unpack_from("<HH", elf, 0x3A)
    for i in range(shnum):
        base = shoff + i * shentsize
        kind, = struct.unpack_from("<I", elf, base + 4)
        off, size = struct.unpack_from("<QQ", elf, base + 24)
        if kind != 7:  # SHT_NOTE
            continue
        end = off + size
        while off < end:
            namesz, descsz, ntype = struct.unpack_from("<III", elf, off)
            off += 12 + (namesz + 3) // 4 * 4
            yield ntype, bytes(elf[off:off + descsz])
            off += (descsz + 3) // 4 * 4


@pytest.fixture(scope="module")
def kernels():
    """{mangled name: metadata} of every kernel in the library."""
    if not os.path.exists(LIB):
        pytest.fail("libintattn.so is not built")
    data = open(LIB, "rb").read()
    out = {}
    for m in re.finditer(rb"__CLANG_OFFLOAD_BUNDLE__", data):
        base = m.start()
        count, = struct.unpack_from("<Q", data, base + 24)
        pos = base + 32
        for _ in range(count):
            off, size, idlen = struct.unpack_from("<QQQ", data, pos)
            target = data[pos + 24:pos + 24 + idlen]
            pos += 24 + idlen
            if b"gfx950" in target and size:
                for ntype, desc in notes(memoryview(data)[base + off:base + off + size]):
                    if ntype == NT_AMDGPU_METADATA:
                        for k in msgpack.unpackb(desc)["amdhsa.kernels"]:
                            out[k[".name"]] = k
    assert len(out) > 50
    return out


def pick(kernels, pattern):
    found = {n: k for n, k in kernels.items() if re.search(pattern, n)}
    assert found, pattern
    return found


def registers(kernels, pattern):
    return max(k[".vgpr_count"] for k in pick(kernels, pattern).values())


@pytest.mark.parametrize("d, most", [(64, 140), (128, 224)])
def test_tiled_kernels_with_sweep_c_on_known_schemes(kernels, d, most):
    """All sweeps, and sweep C alone, of 32 rows a wave on host scales (index schemes 0 to 3)."""
    for phase in (0, 2):
        assert registers(kernels, rf"fwd_kernelILi{d}ELi1ELi2ELb[01]ELi[0-3]ELi{phase}E") <= most


def test_sweep_c_at_head_dimension_64_runs_three_waves(kernels):
    """168 registers a lane let three waves share a SIMD."""
    assert registers(kernels, r"sweep_c_kernelILi64E") <= 168


def test_derivation_kernels_use_no_scratch(kernels):
    assert all(k[".private_segment_fixed_size"] == 0 for k in pick(kernels, r"derive_").values())


def test_row_maxima_alone_have_no_index_map(kernels):
    """Sweep A over a range of the keys: one kernel for each head dimension and mask."""
    assert len(pick(kernels, r"fwd_kernelILi\d+ELi2ELi2ELb[01]ELi\d+ELi3E")) == 4


def test_kernels_with_the_keys_split_over_waves_spill_little(kernels):
    """Row groups and host scales (key groups at d = 128 are at the limit of 256 registers)."""
    assert all(k[".vgpr_spill_count"] <= 10 for k in pick(kernels, r"fwd_splitk_kernelILi\d+ELb[01]ELi[0-6]E").values())
