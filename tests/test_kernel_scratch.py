"""Scratch of the built kernels, read from the library's own gfx950 code
objects: registers that do not fit go to scratch memory, and their reloads wait
for every tile load in flight, so the kernels of the main path use none."""
import re
import struct

import msgpack
import pytest

from paper_2609_37852_amd import binding


def _kernels():
    """name -> metadata of every kernel (the AMDGPU metadata note, a msgpack
    map, of each code object in the library's offload bundles)."""
    b, out, pos = open(binding.LIB_PATH, "rb").read(), {}, 0
    while (pos := b.find(b"__CLANG_OFFLOAD_BUNDLE__", pos)) >= 0:
        entry = pos + 32
        for _ in range(struct.unpack_from("<Q", b, pos + 24)[0]):
            off, size, n = struct.unpack_from("<3Q", b, entry)
            if b"gfx950" in b[entry + 24:entry + 24 + n]:
                elf = b[pos + off:pos + off + size]
                table, = struct.unpack_from("<Q", elf, 0x28)
                width, count = struct.unpack_from("<HH", elf, 0x3A)
                for s in range(count):
                    head = table + width * s
                    at, = struct.unpack_from("<Q", elf, head + 0x18)
                    if struct.unpack_from("<I", elf, head + 4)[0] != 7:      # SHT_NOTE
                        continue
                    namesz, descsz, kind = struct.unpack_from("<3I", elf, at)
                    if kind == 32:                                           # NT_AMDGPU_METADATA
                        at += 12 + (namesz + 3) // 4 * 4
                        meta = msgpack.unpackb(elf[at:at + descsz])
                        out.update((k[".name"], k) for k in meta["amdhsa.kernels"])
            entry += 24 + n
        pos += 24
    return out


# kernel, template arguments in its mangled name, bytes of scratch a lane
@pytest.mark.parametrize("pattern,limit", [
    (r"fwd_kernel\w*ELb[01]ELi1EE", 0),                       # one isolated channel
    (r"fwd_kernel\w*ELb[01]ELi3EE", 32),                      # three: 192 / 128
    (r"delta_matching_kernel\w*ELb[01]ELb[01]ELi[13]ELi1EE", 0),
    (r"delta_matching_kernel\w*ELb[01]ELb[01]ELi[13]ELi2EE", 32),   # two query blocks per wave, d = 128: outside its loops
    (r"bwd_kernelILi\d+ELi\d+ELb0E", 0),                      # without row statistics
    (r"bwd_kernelILi\d+ELi\d+ELb1E", 256),                    # the instrumented one
    (r"(dq|bwd_prep|bwd_reduce|pack_bf16|quantize|stale_rowsum|fill_zero|producer_\w+)_kernel", 0),
])
def test_scratch(pattern, limit):
    found = {n: k[".private_segment_fixed_size"] for n, k in _kernels().items() if re.search(pattern, n)}
    assert found, "no such kernel"
    over = {n: s for n, s in found.items() if s > limit}
    assert not over, over
