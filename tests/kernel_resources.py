"""What the built library's kernels ask of a compute unit, read from the metadata that hipcc leaves in it."""
import struct

import msgpack

MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _code_objects(image):
    at = image.find(MAGIC)
    while at >= 0:
        (n,) = struct.unpack_from("<Q", image, at + len(MAGIC))
        pos = at + len(MAGIC) + 8
        for _ in range(n):
            offset, size, name_len = struct.unpack_from("<QQQ", image, pos)
            name = image[pos + 24:pos + 24 + name_len]
            pos += 24 + name_len
            if b"gfx950" in name:
                yield image[at + offset:at + offset + size]
        at = image.find(MAGIC, at + 1)


def kernels(lib_path):
    """name -> dict with .vgpr_count, .agpr_count, .vgpr_spill_count, .group_segment_fixed_size (bytes of LDS) ..."""
    out = {}
    with open(lib_path, "rb") as f:
        image = f.read()
    for elf in _code_objects(image):
        (sh_off,) = struct.unpack_from("<Q", elf, 0x28)
        sh_size, sh_n = struct.unpack_from("<HH", elf, 0x3A)
        for i in range(sh_n):
            kind, _, _, offset, size = struct.unpack_from("<IQQQQ", elf, sh_off + i * sh_size + 4)
            if kind != 7:                                                # notes
                continue
            name_len, desc_len, note = struct.unpack_from("<III", elf, offset)
            if note == 32:                                               # AMDGPU metadata
                start = offset + 12 + (name_len + 3) // 4 * 4
                for k in msgpack.unpackb(elf[start:start + desc_len])["amdhsa.kernels"]:
                    out[k[".name"]] = k
    return out
