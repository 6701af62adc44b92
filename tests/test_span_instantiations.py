"""The timing aid times the kernel that production runs: an instantiation that takes spans has the registers of its
plain twin and spills no more than it.  Read from the metadata of the built library's gfx950 code."""
import os
import re
import struct

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2401_18079_amd", "libkvq.so")
SHT_NOTE, NT_AMDGPU_METADATA = 7, 32


def _notes(elf):
    shoff, = struct.unpack_from("<Q", elf, 40)
    size, count = struct.unpack_from("<HH", elf, 58)
    for i in range(count):
        kind, = struct.unpack_from("<I", elf, shoff + i * size + 4)
        at, length = struct.unpack_from("<QQ", elf, shoff + i * size + 24)
        end = at + length
        while kind == SHT_NOTE and at < end:
            n_name, n_desc, note = struct.unpack_from("<III", elf, at)
            desc = at + 12 + (n_name + 3) // 4 * 4
            if note == NT_AMDGPU_METADATA:
                yield elf[desc:desc + n_desc]
            at = desc + (n_desc + 3) // 4 * 4


def _kernels():
    msgpack = pytest.importorskip("msgpack")
    with open(LIB, "rb") as f:
        data = f.read()
    magic, out = b"__CLANG_OFFLOAD_BUNDLE__", {}
    at = data.find(magic)
    while at >= 0:                            # one bundle per source file
        entries, = struct.unpack_from("<Q", data, at + 24)
        p = at + 32
        for _ in range(entries):
            offset, size, n = struct.unpack_from("<QQQ", data, p)
            target = data[p + 24:p + 24 + n]
            p += 24 + n
            if b"gfx950" in target and size:
                for note in _notes(data[at + offset:at + offset + size]):
                    for k in msgpack.unpackb(note)["amdhsa.kernels"]:
                        out[k[".name"]] = k
        at = data.find(magic, at + 1)
    return out


def test_timed_kernels_are_the_plain_ones():
    if not os.path.exists(LIB):
        pytest.skip("library not built")
    kernels = _kernels()
    pairs = []
    for name, k in kernels.items():
        m = re.match(r"(.*(?:kvq_qk_kernel|kvq_qkg_kernel|kvq_pv_dense)I.*E)Lb1E(EEv.*)$", name)
        if m:
            pairs.append((k, kernels[m.group(1) + "Lb0E" + m.group(2)]))
    assert len(pairs) > 50
    for timed, plain in pairs:
        # two scalar registers hold the start time; a spill or two may fall differently
        assert timed[".vgpr_spill_count"] <= plain[".vgpr_spill_count"] + 2, timed[".name"]
        assert timed[".private_segment_fixed_size"] <= plain[".private_segment_fixed_size"] + 8, timed[".name"]
        assert timed[".vgpr_count"] <= plain[".vgpr_count"] + 4, timed[".name"]


def test_timed_shared_launches_are_the_plain_ones():
    """Likewise the launch that holds the sparse and dense Value kernels (its span flag is not the last argument)."""
    if not os.path.exists(LIB):
        pytest.skip("library not built")
    kernels = _kernels()
    pairs = []
    for name, k in kernels.items():
        m = re.match(r"(.*kvq_pv_bothILi\dELi\dELb[01]E)Lb1E(.*)$", name)
        if m:
            pairs.append((k, kernels[m.group(1) + "Lb0E" + m.group(2)]))
    assert len(pairs) == 48
    for timed, plain in pairs:
        assert timed[".vgpr_spill_count"] <= plain[".vgpr_spill_count"] + 2, timed[".name"]
        assert timed[".private_segment_fixed_size"] <= plain[".private_segment_fixed_size"] + 8, timed[".name"]
        assert timed[".vgpr_count"] <= plain[".vgpr_count"] + 4, timed[".name"]
