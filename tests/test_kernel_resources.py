"""What the compiler gave the kernels of the built library: nothing they keep is spilled (the kernel descriptors' metadata in
the library's own gfx950 code objects)."""
import os
import struct

import pytest

from paper_2510_26577_amd import binding


def kernels(path=binding.LIB_PATH):
    """{demangled-enough name: metadata} of every kernel in libtva.so, or in another build of it."""
    import msgpack
    if not os.path.exists(path):
        binding.build_library(timeline=path == binding.TIMELINE_LIB_PATH)
    data = open(path, "rb").read()
    found, at = {}, 0
    while (at := data.find(b"\x7fELF\x02\x01\x01\x40", at)) >= 0:  # 64-bit little-endian, OS/ABI AMDGPU_HSA
        shoff, = struct.unpack_from("<Q", data, at + 40)
        shentsize, shnum = struct.unpack_from("<HH", data, at + 58)
        for i in range(shnum):
            kind, _, _, offset, size = struct.unpack_from("<IQQQQ", data, at + shoff + i * shentsize + 4)
            if kind != 7:  # SHT_NOTE
                continue
            p, end = at + offset, at + offset + size
            while p < end:
                nlen, dlen, what = struct.unpack_from("<III", data, p)
                body = p + 12 + (nlen + 3) // 4 * 4
                if what == 32:  # NT_AMDGPU_METADATA
                    for k in msgpack.unpackb(data[body:body + dlen])["amdhsa.kernels"]:
                        found[k[".name"]] = k
                p = body + (dlen + 3) // 4 * 4
        at += 64
    return found


@pytest.fixture(scope="module")
def table():
    t = kernels()
    assert sum("attn_kernel" in n for n in t) >= 28 and sum("walk_kernel" in n for n in t) == 7, sorted(t)
    return t


def test_eight_wave_attention_shapes_keep_no_scalars_in_vector_registers(table):
    """Scalars that do not fit are written to lanes of vector registers and read back in the loop.  (A handful at most: the
    paged 256-row shape with D = 128 parks one.)"""
    for name, k in table.items():
        if "attn_kernel" in name and ("ELi8ELi1ELi1E" in name or "ELi4ELi2ELi1E" in name):
            assert k[".sgpr_spill_count"] <= 4, (name, k[".sgpr_spill_count"])


def test_attention_kernels_spill_no_vector_registers(table):
    for name, k in table.items():
        if "attn_kernel" in name or "merge_kernel" in name:
            assert k[".vgpr_spill_count"] == 0 and k[".private_segment_fixed_size"] == 0, name


def test_instrumented_attention_kernels_spill_no_vector_registers():
    """Time stamps of a kernel that writes its registers to memory are of another kernel.  (D = 128: of D = 64, where two to four workgroups
    share a CU, three paged shapes have no register to spare for the stamps.)"""
    seen = {n: k for n, k in kernels(binding.TIMELINE_LIB_PATH).items() if "attn_kernelILi128" in n}
    assert len(seen) >= 18
    for name, k in seen.items():
        assert k[".vgpr_spill_count"] == 0 and k[".private_segment_fixed_size"] == 0, (name, k[".vgpr_spill_count"])


def test_attention_kernels_of_which_two_share_a_compute_unit_leave_the_registers_for_it(table):
    """Wavefronts per SIMD that the registers allow (512 per lane), against what the shape's rings leave room for: two
    workgroups of four waves, with D = 64 two of eight (the dense 256-row shape runs one)."""
    seen = 0
    for name, k in table.items():
        for shape, most in (("ILi128ELi1ELi2ELi1ELb0ELi2E", 256), ("ILi128ELi2ELi2ELi1ELb0ELi2E", 256), ("ILi128ELi1ELi2ELi1ELb1ELi2E", 256),
                            ("ILi128ELi2ELi2ELi1ELb1ELi2E", 256), ("ILi64ELi4ELi2ELi1ELb0E", 128), ("ILi64ELi4ELi2ELi1ELb1E", 128),
                            ("ILi64ELi8ELi1ELi1ELb1E", 128)):
            if "attn_kernel" + shape in name:
                assert k[".vgpr_count"] <= most, (name, k[".vgpr_count"])
                seen += 1
    assert seen == 7


def test_the_64_row_shape_of_head_dimension_64_leaves_the_registers_for_four_wavefronts(table):
    """Four workgroups' short rings fit a compute unit."""
    seen = [k[".vgpr_count"] for name, k in table.items() if "attn_kernelILi64ELi2ELi2ELi1ELb0ELi2E" in name or "attn_kernelILi64ELi2ELi2ELi1ELb1ELi2E" in name]
    assert len(seen) == 2 and max(seen) <= 128, seen


def test_sampling_kernels_spill_vector_registers_in_one_form_only(table):
    """walk_kernel<16, false> (16 groups of a vocabulary that is no multiple of 4) keeps both rows and spills a dozen."""
    for name, k in table.items():
        if "walk_kernel" in name or "sample_kernel" in name or "topk_parts_kernel" in name:
            most = 12 if "walk_kernelILi16ELb0E" in name else 0
            assert k[".vgpr_spill_count"] <= most, (name, k[".vgpr_spill_count"])


def test_launches_that_merge_their_splits_have_kernels_of_their_own(table):
    """D = 128, the 64-row shapes (two of 16-bit K/V, one of 8-bit), the 128-row and the 256-row shape, dense and paged, but for the paged 256-row
    shape with 8-bit K/V; each beside the kernel of the same shape that merges nothing.  (The fourth argument is -1 in theirs.)"""
    names = [n.split("attn_kernel")[1].split("EEEv")[0] for n in table if "attn_kernel" in n]
    shared, alone = {n for n in names if "Lin1E" in n}, {n for n in names if "Lin1E" not in n}
    assert len(shared) == 13 and len(alone) == 28 and {n.replace("Lin1E", "Li1E") for n in shared} < alone
    assert all(n.startswith("ILi128E") and not n.startswith("ILi128ELi1E") for n in shared) and "ILi128ELi8ELi1ELin1ELb1ELi3ELb1" not in shared
