"""What the compiler gave the library's kernels, from the code objects' own metadata: registers that do not suffice go to scratch
memory, and nothing in a result shows it."""
import os
import struct

import msgpack

import paper_2508_11584_amd as vpe

LIB = os.path.join(os.path.dirname(os.path.abspath(vpe.__file__)), "libvpe.so")


def kernels():
    """The metadata of every gfx950 kernel: the offload bundles' code objects, each with one AMDGPU note in msgpack."""
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
                note = code.find(b"AMDGPU\0\0")
                out += msgpack.unpackb(code[note + 8:note + 8 + struct.unpack_from("<I", code, note - 8)[0]])["amdhsa.kernels"]
            p += 24 + length
        at += len(magic)
    return out


def test_no_kernel_keeps_registers_in_scratch_memory():
    found = kernels()
    assert sum("gemm_dma_kernel" in k[".name"] for k in found) > 50 and any("attention_kernel" in k[".name"] for k in found)
    spilled = [(k[".name"], k[".vgpr_spill_count"], k[".private_segment_fixed_size"]) for k in found
               if k[".vgpr_spill_count"] or k[".private_segment_fixed_size"]]
    assert not spilled, spilled


def test_scalar_registers_of_the_kernels():
    # (what a spilled scalar register costs depends on where it is read: the attention kernels may keep up to 32 for what follows
    # their key loop; with an iteration's load addresses among them they kept 67 and 149, read back in every iteration)
    spilled = {k[".name"]: k[".sgpr_spill_count"] for k in kernels() if k[".sgpr_spill_count"]}
    assert all("attention_kernel" in name and n <= 32 for name, n in spilled.items()), spilled
