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


# Index schemes (the fifth template argument): 0 double, 4 every head its own, 5 row groups, 7 key groups, 9 fma.
@pytest.mark.parametrize("d, schemes, most", [(64, "[49]", 144), (64, "[05]", 128), (128, "[0459]", 224)])
def test_tiled_kernels_with_sweep_c(kernels, d, schemes, most):
    """All sweeps, and sweep C alone, of 32 rows a wave.  A SIMD holds four waves up to 128 registers a lane, three up to 168,
    two up to 256."""
    for phase in (0, 2):
        assert registers(kernels, rf"fwd_kernelILi{d}ELi1ELi2ELb[01]ELi{schemes}ELi{phase}E") <= most


@pytest.mark.parametrize("d, most", [(64, 128), (128, 168)])
def test_sweep_c_runs_three_or_four_waves(kernels, d, most):
    """Spills, of two to four registers, only where the double map is held in sweep C of unsplit keys."""
    assert registers(kernels, rf"sweep_c_kernelILi{d}E") <= most
    for name, k in pick(kernels, rf"sweep_c_kernelILi{d}ELb[01]ELi[0459]ELb[01]E").items():
        assert k[".vgpr_spill_count"] <= (4 if re.search(r"Li128ELb[01]ELi[04]ELb0E", name) else 0), name


@pytest.mark.parametrize("d, rows, most, spilled", [(64, 1, 128, 0), (128, 1, 128, 0), (128, 2, 168, 14)])
def test_sweeps_a_and_b_run_three_or_four_waves(kernels, d, rows, most, spilled):
    """Two blocks of rows a wave hold three waves a SIMD at the price of 3 to 5 spilled registers with the fma map, up to 13
    where the kernel holds both maps."""
    found = pick(kernels, rf"fwd_kernelILi{d}ELi{rows}ELi2ELb[01]ELi[0459]ELi1E")
    assert max(k[".vgpr_count"] for k in found.values()) <= most
    assert max(k[".vgpr_spill_count"] for k in found.values()) <= spilled
    assert all(k[".vgpr_spill_count"] <= 5 for n, k in found.items() if "ELi9E" in n)


def test_sweep_b_over_a_range_of_keys(kernels):
    assert registers(kernels, r"fwd_kernelILi\d+ELi2ELi2ELb[01]ELi[0459]ELi4E") <= 168
    assert all(k[".vgpr_spill_count"] <= 8 for k in pick(kernels, r"fwd_kernelILi\d+ELi2ELi2ELb[01]ELi[0459]ELi4E").values())


def test_short_sequences_run_three_waves(kernels):
    """All scores in registers: 168 a lane for up to 256 keys, 128 for up to 128."""
    assert registers(kernels, r"fwd_short_kernelILi[478]E") <= 168
    assert registers(kernels, r"fwd_short_kernelILi4E") <= 128


def test_derivation_kernels_use_no_scratch(kernels):
    assert all(k[".private_segment_fixed_size"] == 0 for k in pick(kernels, r"derive_").values())


def test_row_maxima_alone_have_no_index_map(kernels):
    """Sweep A over a range of the keys: one kernel for each head dimension and mask."""
    assert len(pick(kernels, r"fwd_kernelILi\d+ELi2ELi2ELb[01]ELi\d+ELi3E")) == 4


def test_kernels_with_the_keys_split_over_waves_do_not_spill(kernels):
    """Two waves a SIMD at d = 128, three at d = 64 (key groups: two)."""
    found = pick(kernels, r"fwd_splitk_kernelILi\d+ELb[01]ELi[04579]E")
    assert len(found) == 28 and all(k[".vgpr_spill_count"] == 0 for k in found.values())
    assert registers(kernels, r"fwd_splitk_kernelILi64ELb[01]ELi[0459]E") <= 168
