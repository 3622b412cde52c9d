"""What the compiler made of the kernels, from the metadata of the library's own code objects: kernels whose speed hangs on their
registers neither spill nor take more than their workgroups share a CU with."""
import os
import re
import struct

import pytest

msgpack = pytest.importorskip("msgpack")

LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2306_06446_amd", "libshiftadd.so")


def kernel_metadata(elf):
    """name -> metadata of every kernel of a code object (its AMDGPU metadata note, a msgpack map)."""
    shoff, = struct.unpack_from("<Q", elf, 40)
    entry, count = struct.unpack_from("<HH", elf, 58)
    found = {}
    for i in range(count):
        _, kind, _, _, at, size = struct.unpack_from("<IIQQQQ", elf, shoff + i * entry)
        end = at + size
        while kind == 7 and at < end:                        # SHT_NOTE
            name_size, desc_size, note = struct.unpack_from("<III", elf, at)
            desc = at + 12 + (name_size + 3) // 4 * 4
            if note == 32:                                   # NT_AMDGPU_METADATA
                meta = msgpack.unpackb(elf[desc:desc + desc_size], strict_map_key=False)
                found.update({k[".name"]: k for k in meta["amdhsa.kernels"]})
            at = desc + (desc_size + 3) // 4 * 4
    return found


@pytest.fixture(scope="module")
def kernels():
    if not os.path.exists(LIB):
        import __graft_entry__
        __graft_entry__.build()
    data, found, at = open(LIB, "rb").read(), {}, 0
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    while True:
        at = data.find(magic, at)
        if at < 0:
            return found
        count, = struct.unpack_from("<Q", data, at + len(magic))
        p = at + len(magic) + 8
        for _ in range(count):
            offset, size, length = struct.unpack_from("<QQQ", data, p)
            target = data[p + 24:p + 24 + length]
            p += 24 + length
            if size and b"gfx950" in target:
                found.update(kernel_metadata(data[at + offset:at + offset + size]))
        at += len(magic)


@pytest.mark.parametrize("pattern,instances", [
    (r"qkv_mfma_kernel", 24),
    (r"ktv_mfma_kernel|ktv_qkv_kernel", 28),
    (r"norm_linear_kernel", 4),
    (r"gemm_kernel.*HashStore", 8),
    (r"linear_norm_kernel", 3),
    (r"shift_mlp_kernel", 21),
    (r"shift_mlp_walk_kernel", 3),
    (r"norm_hash_kernel", 32),
    (r"hamming_pipe_kernel", 6),
    (r"gemm_kernel.*ShiftStoreILi6E|gemm_even_kernel.*ShiftStoreILi6E", 15),      # fp32 Linears with a residual, or into Q, K and V
    (r"decode_works?_kernel|decode_w4_kernel|side_work_kernel", 4),      # a choice of argument by lane keeps the arguments in scratch
])
def test_no_scratch(kernels, pattern, instances):
    some = {n: k for n, k in kernels.items() if re.search(pattern, n)}
    assert len(some) == instances
    for n, k in some.items():
        assert k[".private_segment_fixed_size"] == 0 and k[".vgpr_spill_count"] == 0, n


# two workgroups of eight wavefronts to a CU: K^T V, alone or with Q(K^T V), for many short sequences (a ring of two), and others
@pytest.mark.parametrize("pattern,instances", [
    (r"ktv_qkv_kernelILi\d+ELi\d+ELi\d+ELi\d+ELi2EE", 4),
    (r"ktv_mfma_kernelILi\d+ELi\d+ELi\d+ELi2ELb[01]EE", 8),
    (r"norm_hash_kernelILi1ELi32ELi64ELb0EE", 1),           # rows of 64 columns, heads of 32
    (r"hamming_pipe_kernel", 6),
])
def test_registers_for_two_workgroups(kernels, pattern, instances):
    some = {n: k for n, k in kernels.items() if re.search(pattern, n)}
    assert len(some) == instances
    for n, k in some.items():
        assert k[".vgpr_count"] <= 128, n


# the LayerNorm of 4097 to 8192 columns holds a row on 64 lanes, more than they have registers for
def test_no_other_kernel_has_scratch(kernels):
    spilled = {n for n, k in kernels.items() if k[".private_segment_fixed_size"] or k[".vgpr_spill_count"]}
    assert len(kernels) > 350
    assert all(re.search(r"layernorm_kernelILi64ELi32E", n) for n in spilled) and len(spilled) == 2, spilled


# a CU's two or three workgroups of both experts' tiles, and its four, two or one of few rows
@pytest.mark.parametrize("pattern,instances,registers,lds", [
    (r"expert_split_kernel", 5, 256, 80 * 1024),
    (r"expert_even_kernel", 2, 168, 160 * 1024 // 3),
    (r"gemm_even_kernel", 10, 168, 160 * 1024 // 3),
    (r"few_rows_kernelILi1ELi1E", 4, 128, 40 * 1024),
    (r"few_rows_kernelILi2ELi1E", 4, 128, 80 * 1024),
    (r"few_rows_kernelILi3ELi1E", 4, 80, 80 * 1024),         # 24 wavefronts
    (r"few_rows_kernelILi4ELi1E|few_rows_kernelILi[34]ELi[24]E", 9, 128, 160 * 1024),
])
def test_workgroups_that_share_a_cu(kernels, pattern, instances, registers, lds):
    some = {n: k for n, k in kernels.items() if re.search(pattern, n)}
    assert len(some) == instances
    for n, k in some.items():
        assert k[".vgpr_count"] <= registers and k[".group_segment_fixed_size"] <= lds, n
