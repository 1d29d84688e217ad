"""What the compiler gave the library's kernels, from the code objects' own metadata: registers that do not suffice go to scratch
memory, and nothing in a result shows it."""
import os
import struct

import paper_2508_11584_amd as vpe

LIB = os.path.join(os.path.dirname(os.path.abspath(vpe.__file__)), "libvpe.so")
SIZES = {0xCC: ">B", 0xCD: ">H", 0xCE: ">I", 0xD9: ">B", 0xDA: ">H"}        # MessagePack: unsigned integers, strings


def values(code, key):
    """What follows every occurrence of a key in the AMDGPU note's MessagePack: a small unsigned integer or a string."""
    out, at = [], 0
    while (at := code.find(key, at)) >= 0:
        at += len(key)
        tag, p = code[at], at + 1
        if tag in SIZES:
            number, = struct.unpack_from(SIZES[tag], code, p)
            p += struct.calcsize(SIZES[tag])
        else:
            number = tag & (0x1F if tag >= 0xA0 else 0x7F)
        out.append(code[p:p + number].decode() if tag in (0xD9, 0xDA) or 0xA0 <= tag < 0xC0 else number)
    return out


def kernels():
    """(symbol, vector spills, scalar spills, bytes of scratch a lane) of every gfx950 kernel, from the offload bundles' code objects."""
    vpe.load_library()
    with open(LIB, "rb") as f:
        data = f.read()
    magic, out, at = b"__CLANG_OFFLOAD_BUNDLE__", [], 0
    while (at := data.find(magic, at)) >= 0:
        entries, p = struct.unpack_from("<Q", data, at + 24)[0], at + 32
        for _ in range(entries):
            offset, size, length = struct.unpack_from("<QQQ", data, p)
            if b"gfx950" in data[p + 24:p + 24 + length]:
                code = data[at + offset:at + offset + size]
                columns = [values(code, k) for k in (b".symbol", b".vgpr_spill_count", b".sgpr_spill_count", b".private_segment_fixed_size")]
                assert len({len(c) for c in columns}) == 1          # (a unit without kernels has none of them)
                out += zip(*columns)
            p += 24 + length
        at += len(magic)
    return out


def test_no_kernel_keeps_registers_in_scratch_memory():
    found = kernels()
    assert sum("gemm_dma_kernel" in name for name, *_ in found) > 50 and any("attention_kernel" in name for name, *_ in found)
    spilled = [(name, vector, scratch) for name, vector, _, scratch in found if vector or scratch]
    assert not spilled, spilled


def test_scalar_registers_of_the_kernels():
    # (what a spilled scalar register costs depends on where it is read: the attention kernels may keep up to 32 for what follows
    # their key loop; with an iteration's load addresses among them they kept 67 and 149, read back in every iteration)
    spilled = {name: scalar for name, _, scalar, _ in kernels() if scalar}
    assert all("attention_kernel" in name and n <= 32 for name, n in spilled.items()), spilled
