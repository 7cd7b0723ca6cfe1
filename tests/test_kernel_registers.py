"""What the compiler made of the grouped FFN's kernels, read from the metadata of the built library: no vector register in
memory.  (Its waits count memory operations by hand, and a reload waits for every store issued before it.)"""
import struct

import msgpack

from paper_2411_10003_amd import binding


def _kernels(path):
    """Metadata of every gfx950 kernel: the offload bundles of the library, the notes of their ELF files."""
    data, out, at = open(path, "rb").read(), [], 0
    while (at := data.find(b"__CLANG_OFFLOAD_BUNDLE__", at)) >= 0:
        p = at + 32
        for _ in range(struct.unpack_from("<Q", data, at + 24)[0]):
            off, size, n = struct.unpack_from("<QQQ", data, p)
            triple, p = data[p + 24:p + 24 + n], p + 24 + n
            if b"gfx950" not in triple:
                continue
            elf = data[at + off:at + off + size]
            sections, (entry, count) = struct.unpack_from("<Q", elf, 0x28)[0], struct.unpack_from("<HH", elf, 0x3A)
            for i in range(count):
                _, kind, _, _, o, end = struct.unpack_from("<IIQQQQ", elf, sections + i * entry)
                end += o
                while kind == 7 and o < end:                   # SHT_NOTE; NT_AMDGPU_METADATA
                    name, desc, note = struct.unpack_from("<III", elf, o)
                    o += 12 + (name + 3) // 4 * 4
                    if note == 32:
                        out += msgpack.unpackb(elf[o:o + desc])["amdhsa.kernels"]
                    o += (desc + 3) // 4 * 4
        at += 8
    return out


def test_grouped_ffn_keeps_its_registers():
    kernels = [k for k in _kernels(binding.LIB_PATH) if "grouped_gemm_kernel" in k[".name"]]
    assert len(kernels) >= 32, len(kernels)
    spilled = {k[".name"]: (k[".vgpr_spill_count"], k[".private_segment_fixed_size"]) for k in kernels
               if k[".vgpr_spill_count"] or k[".private_segment_fixed_size"]}
    assert not spilled, spilled
