"""What the compiler gave the kernels, read from the metadata of the built library's code objects: no kernel of a plain call may pass
values through scratch memory (a round trip each, in chains whose round trips are what a short call takes)."""
import os
import re
import struct

import msgpack
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def code_objects(lib):
    """The gfx950 code objects of the library: entries of its offload bundles."""
    for m in re.finditer(b"__CLANG_OFFLOAD_BUNDLE__", lib):
        at = m.end()
        (n,) = struct.unpack_from("<Q", lib, at)
        at += 8
        for _ in range(n):
            off, size, idlen = struct.unpack_from("<QQQ", lib, at)
            name = lib[at + 24:at + 24 + idlen]
            at += 24 + idlen
            if b"gfx950" in name:
                yield lib[m.start() + off:m.start() + off + size]


def kernels(elf):
    """The entries of `amdhsa.kernels` in the code object's metadata note."""
    shoff, = struct.unpack_from("<Q", elf, 0x28)
    size, count = struct.unpack_from("<HH", elf, 0x3A)
    for i in range(count):
        kind, = struct.unpack_from("<I", elf, shoff + i * size + 4)
        if kind != 7:   # SHT_NOTE
            continue
        at, length = struct.unpack_from("<QQ", elf, shoff + i * size + 0x18)
        end = at + length
        while at + 12 <= end:
            nlen, dlen, ntype = struct.unpack_from("<III", elf, at)
            body = at + 12 + (nlen + 3) // 4 * 4
            if ntype == 32:   # NT_AMDGPU_METADATA
                yield from msgpack.unpackb(elf[body:body + dlen])["amdhsa.kernels"]
            at = body + (dlen + 3) // 4 * 4


@pytest.fixture(scope="module")
def table():
    with open(os.path.join(ROOT, "paper_2409_16546_amd", "libakv.so"), "rb") as f:
        lib = f.read()
    t = {k[".name"]: k for o in code_objects(lib) for k in kernels(o)}
    assert len(t) > 50
    return t


def test_no_kernel_of_a_plain_call_uses_scratch_memory(table):
    # the variants that export masks and counters (head_kernel<1, NT, true, ...>) have the register limit of the plain ones and may spill
    exports = re.compile(r"head_kernelILi1ELi\d+ELb1E")
    bad = {n: k[".private_segment_fixed_size"] for n, k in table.items() if k[".private_segment_fixed_size"] and not exports.search(n)}
    assert not bad


def test_four_workgroups_of_the_selection_kernel_share_a_compute_unit(table):
    """One workgroup per query head: calls of many heads run them in rounds.  A SIMD has 512 vector registers per lane and 800 scalar ones, a unit
    160 KB of LDS."""
    variants = [k for n, k in table.items() if "split_select_kernelILi512E" in n]
    assert variants
    for k in variants:
        waves = k[".max_flat_workgroup_size"] // 64   # per SIMD: those of four workgroups on four SIMDs
        assert (k[".vgpr_count"] + 7) // 8 * 8 * waves <= 512 and k[".sgpr_count"] * waves <= 800
        assert 4 * k[".group_segment_fixed_size"] <= 160 * 1024


def test_four_workgroups_of_the_short_k_kernel_share_a_compute_unit(table):
    """Up to six workgroups of four waves per unit: a wave per SIMD each."""
    variants = [k for n, k in table.items() if "split_k_short_kernel" in n]
    assert len(variants) == 4
    for k in variants:
        assert k[".vgpr_count"] <= 128 and 4 * k[".group_segment_fixed_size"] <= 160 * 1024
