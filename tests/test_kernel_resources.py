"""What the compiler gave the prompt's kernels, from the metadata of the built library."""
import re
import struct

import pytest

from paper_2505_10938_amd import binding as B

msgpack = pytest.importorskip("msgpack")


def kernels():
    """Metadata of every kernel of libkvq.so, by its mangled name."""
    data = open(B.LIB_PATH, "rb").read()
    out = {}
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    at = data.find(magic)
    while at >= 0:                                            # one bundle per source file
        count, = struct.unpack_from("<Q", data, at + 24)
        p = at + 32
        for _ in range(count):
            offset, size, n = struct.unpack_from("<QQQ", data, p)
            if b"gfx950" in data[p + 24:p + 24 + n]:
                out.update(notes(data[at + offset:at + offset + size]))
            p += 24 + n
        at = data.find(magic, p)
    return out


def notes(elf):
    first, = struct.unpack_from("<Q", elf, 32)
    entry, count = struct.unpack_from("<HH", elf, 54)
    for i in range(count):
        kind, = struct.unpack_from("<I", elf, first + i * entry)
        offset, _, _, size = struct.unpack_from("<QQQQ", elf, first + i * entry + 8)
        p, end = offset, offset + size
        while kind == 4 and p < end:                          # PT_NOTE
            name, desc, tag = struct.unpack_from("<III", elf, p)
            body = p + 12 + (name + 3) // 4 * 4
            if tag == 32 and elf[p + 12:p + 18] == b"AMDGPU":
                return {k[".name"]: k for k in msgpack.unpackb(elf[body:body + desc])["amdhsa.kernels"]}
            p = body + (desc + 3) // 4 * 4
    return {}


def test_kernels_of_one_layer_take_the_pointers_of_one():
    """Up to 32 layers have two arrays of 256 bytes in the arguments, one layer two pointers."""
    sizes = {1: [], 32: []}
    for name, kernel in kernels().items():
        if "9LayerRows" in name:
            layers = int(re.search(r"Li(\d+)E(?:Lb\dE)?EEv", name).group(1))
            sizes[layers].append([x[".size"] for x in kernel[".args"] if x[".value_kind"] == "by_value"][-1])
    assert min(map(len, sizes.values())) >= 6 + 6 + 3 + 12 + 1
    assert set(sizes[1]) == {16} and set(sizes[32]) == {512}


@pytest.mark.parametrize("kernel,instances,bytes_of_scratch", [
    ("15quantize_kernelILi", 6, lambda name: 0),
    ("22prompt_quantize_kernelILi", 6, lambda name: 0),
    ("24prompt_candidates_kernelILi", 3, lambda name: 0),
    ("21prompt_compete_kernelILi", 12, lambda name: 0),
])
def test_rows_on_their_way_to_lds_do_not_pass_through_scratch_memory(kernel, instances, bytes_of_scratch):
    found = {n: k[".private_segment_fixed_size"] for n, k in kernels().items() if kernel in n}
    assert len(found) >= instances
    assert found == {n: bytes_of_scratch(n) for n in found}


def test_two_workgroups_that_look_for_candidates_fit_a_compute_unit():
    """1024 threads are four wavefronts per SIMD, whose 512 registers eight share with 64 each."""
    found = {n: k[".vgpr_count"] for n, k in kernels().items() if "24prompt_candidates_kernelILi" in n}
    assert len(found) >= 6 and max(found.values()) <= 64, found
