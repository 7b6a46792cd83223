"""What the compiler's metadata in the built library says of the kernels: nothing that the library launches by its own choice keeps
registers in scratch memory."""
import re
import struct

import msgpack

import paper_2605_29860_amd as espo

MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _code_objects(data):
    for m in re.finditer(re.escape(MAGIC), data):
        at = m.start() + len(MAGIC)
        count, = struct.unpack_from("<Q", data, at)
        at += 8
        for _ in range(count):
            offset, size, idlen = struct.unpack_from("<QQQ", data, at)
            name = data[at + 24:at + 24 + idlen]
            at += 24 + idlen
            if b"gfx950" in name and size:
                yield data[m.start() + offset:m.start() + offset + size]


def _kernels():
    data = open(espo.library_path(), "rb").read()
    for obj in _code_objects(data):
        for m in re.finditer(b"AMDGPU\0\0", obj):             # the note's name, behind its sizes and its type
            namesz, descsz, kind = struct.unpack_from("<III", obj, m.start() - 12)
            if namesz == 7 and kind == 32:
                yield from msgpack.unpackb(obj[m.end():m.end() + descsz])["amdhsa.kernels"]


def test_no_kernel_keeps_registers_in_scratch():
    kernels = {k[".name"]: k for k in _kernels()}
    assert sum("espo_filtered_kernel" in n for n in kernels) == 8 and sum("espo_step_kernel" in n for n in kernels) == 18
    for name, k in kernels.items():
        # workgroups of 4 waves are launched for a forced split only (espo_debug_step), bound to 64 registers
        if "espo_step_kernel" in name and "Li4E" in name:
            continue
        assert k[".private_segment_fixed_size"] == 0 and k[".vgpr_spill_count"] == 0, (name, k[".vgpr_spill_count"])
