"""What the compiler made of the kernels, from the notes in the built library (CPU only)."""
import os
import struct

import msgpack
import pytest

from paper_2605_29639_amd import kvq

AMDGPU_METADATA = 32   # note type of the kernels' metadata, a msgpack map
KNOWN = {"_ZN3kvq12_GLOBAL__N_116attn_rows_kernelILi2ELi128ELb1ELb0EEEvNS_8AttnArgsE": 44,   # bf16, a shared prefix
         "_ZN3kvq12_GLOBAL__N_116attn_wide_kernelILi0EEEvNS_8AttnArgsE": 28}                   # int8, 256 rows


def _notes(elf):
    """(type, descriptor) of all notes of a little-endian 64-bit ELF image."""
    at, = struct.unpack_from("<Q", elf, 32)
    size, count = struct.unpack_from("<HH", elf, 54)
    for i in range(count):
        kind, _, start, _, _, length = struct.unpack_from("<IIQQQQ", elf, at + i * size)
        if kind != 4:   # PT_NOTE
            continue
        end = start + length
        while start + 12 <= end:
            names, descs, note = struct.unpack_from("<III", elf, start)
            start += 12 + (names + 3) // 4 * 4
            yield note, elf[start:start + descs]
            start += (descs + 3) // 4 * 4


def _kernels(path):
    """The metadata of every gfx950 kernel in the library's offload bundles."""
    data, found, at = open(path, "rb").read(), [], 0
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    while (at := data.find(magic, at)) >= 0:
        entries, = struct.unpack_from("<Q", data, at + len(magic))
        p = at + len(magic) + 8
        if entries > 16:   # (the magic's own text elsewhere)
            at += 1
            continue
        for _ in range(entries):
            offset, size, length = struct.unpack_from("<QQQ", data, p)
            target = data[p + 24:p + 24 + length].decode()
            p += 24 + length
            if "gfx950" in target:
                image = data[at + offset:at + offset + size]
                for note, desc in _notes(image):
                    if note == AMDGPU_METADATA:
                        found += msgpack.unpackb(desc)["amdhsa.kernels"]
        at += len(magic)
    return found


@pytest.mark.parametrize("path", [kvq.LIB_PATH, kvq.PROF_LIB_PATH], ids=os.path.basename)
def test_no_kernel_spills_to_memory(path):
    """Registers that do not fit go to scratch memory silently, and what the kernel then waits for is not in the
    source: int8 with two row tiles at head_dim 64 once kept ten there.  (Two kernels that own a SIMD with one or two
    wavefronts keep a few values there outside their loops.)"""
    kernels = _kernels(path)
    assert len({k[".symbol"] for k in kernels}) > 100
    scratch = {k[".name"]: k[".private_segment_fixed_size"] for k in kernels if k[".private_segment_fixed_size"]}
    assert {n: b for n, b in scratch.items() if b > KNOWN.get(n, 0)} == {}
