"""Registers and scratch of the built kernels, from the metadata notes of the
library's own code objects.  A kernel that spills inside its time loop waits
for its prefetched loads at every reload, which no parity test shows."""
import os
import re
import struct

import msgpack
import pytest

from paper_2608_02560_amd import build


def _code_objects(data):
    """The gfx950 ELF images in the library's offload bundles."""
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    at = data.find(magic)
    while at >= 0:
        entry = at + 32
        for _ in range(struct.unpack_from("<Q", data, at + 24)[0]):
            off, size, n = struct.unpack_from("<QQQ", data, entry)
            target = data[entry + 24:entry + 24 + n].decode()
            entry += 24 + n
            if build.ARCH in target:
                yield data[at + off:at + off + size]
        at = data.find(magic, at + len(magic))


def _notes(elf):
    """Descriptors of the AMDGPU metadata notes (type 32) of an ELF image."""
    phoff = struct.unpack_from("<Q", elf, 32)[0]
    size, count = struct.unpack_from("<HH", elf, 54)
    for i in range(count):
        ph = phoff + i * size
        if struct.unpack_from("<I", elf, ph)[0] != 4:  # PT_NOTE
            continue
        at, end = struct.unpack_from("<Q", elf, ph + 8)[0], 0
        end = at + struct.unpack_from("<Q", elf, ph + 32)[0]
        while at < end:
            nlen, dlen, kind = struct.unpack_from("<III", elf, at)
            desc = at + 12 + (nlen + 3 & ~3)
            if kind == 32:
                yield elf[desc:desc + dlen]
            at = desc + (dlen + 3 & ~3)


@pytest.fixture(scope="module")
def kernels():
    if not os.path.exists(build.LIB):
        build.build()
    with open(build.LIB, "rb") as f:
        data = f.read()
    found = {}
    for elf in _code_objects(data):
        for note in _notes(elf):
            for k in msgpack.unpackb(note)["amdhsa.kernels"]:
                found[k[".name"]] = k
    assert len(found) > 300
    return found


def _pick(kernels, pattern):
    got = {n: k for n, k in kernels.items() if re.search(pattern, n)}
    assert got, pattern
    return got


def test_readout_free_scans_keep_their_registers(kernels):
    """bf16 inputs with 16 states a lane, state-only and summary kinds (the
    fifth and seventh template arguments: the kind and the trajectory mode):
    no scratch, and four waves per SIMD."""
    for name, k in _pick(kernels, r"11scan_kernelILi(16|32|64)ENS_6bf16_tEfN?\w*?Li[12]ELb0ELi0EE").items():
        assert k[".private_segment_fixed_size"] == 0 and k[".vgpr_count"] <= 128, name


def test_trajectories_keep_three_waves(kernels):
    for name, k in _pick(kernels, r"11scan_kernelILi(16|32|64)ENS_6bf16_tEfN?\w*?Li1ELb0ELi[12]EE").items():
        assert k[".private_segment_fixed_size"] == 0 and k[".vgpr_count"] <= 168, name


def test_complex_scans_keep_three_waves(kernels):
    for name, k in _pick(kernels, r"19scan_complex_kernelILi16E").items():
        assert k[".private_segment_fixed_size"] == 0 and k[".vgpr_count"] <= 168, name


def test_the_few_query_screen_fits_as_often_as_it_is_launched(kernels):
    """No scratch in the block loop, and registers and LDS for the workgroups of
    four waves per CU that the launch counts on ({prepared, steps}: number)."""
    per_cu = {(1, 2): 4, (1, 8): 4, (1, 16): 2, (0, 2): 4, (0, 8): 3, (0, 16): 2}
    for (prep, steps), n in per_cu.items():
        (k,) = _pick(kernels, r"17screen_few_kernelILb%dELi%dEE" % (prep, steps)).values()
        assert k[".private_segment_fixed_size"] == 0
        assert 512 // (-(-k[".vgpr_count"] // 8) * 8) >= n and 163840 // k[".group_segment_fixed_size"] >= n
