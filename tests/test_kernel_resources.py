"""Register spills of the built kernels, from the metadata the compiler writes into
libsoma.so beside each of them (the code objects' AMDGPU notes): the streaming heads
and projections keep their weights in registers and count on a loop without scratch
accesses, whose loads and stores would stand in the queue of the tiles they stage."""
import os
import re
import struct

import msgpack
import pytest

from paper_2609_37899_amd import soma


def sections(elf):
    off, = struct.unpack_from("<Q", elf, 0x28)
    size, num, names_at = struct.unpack_from("<HHH", elf, 0x3A)
    heads = [struct.unpack_from("<IIQQQQIIQQ", elf, off + i * size) for i in range(num)]
    names = elf[heads[names_at][4]:][:heads[names_at][5]]
    for h in heads:
        yield names[h[0]:names.index(b"\0", h[0])].decode(), h[1], elf[h[4]:h[4] + h[5]] if h[1] != 8 else b""


def code_objects(fat):
    """The gfx code objects of a .hip_fatbin section: bundles of (offset, size, target) entries."""
    magic, at = b"__CLANG_OFFLOAD_BUNDLE__", -1
    while (at := fat.find(magic, at + 1)) >= 0:
        n, = struct.unpack_from("<Q", fat, at + 24)
        p = at + 32
        for _ in range(n):
            off, size, length = struct.unpack_from("<QQQ", fat, p)
            target = fat[p + 24:p + 24 + length]
            p += 24 + length
            if b"gfx950" in target and size:
                yield fat[at + off:at + off + size]


@pytest.fixture(scope="module")
def kernels():
    if not os.path.exists(soma.LIB_PATH):
        from paper_2609_37899_amd import build
        build.build()
    lib = open(soma.LIB_PATH, "rb").read()
    out = {}
    for name, _, fat in sections(lib):
        if name != ".hip_fatbin":
            continue
        for co in code_objects(fat):
            for _, kind, note in sections(co):
                if kind != 7 or struct.unpack_from("<I", note, 8)[0] != 32:   # NT_AMDGPU_METADATA
                    continue
                name_size, size = struct.unpack_from("<II", note, 0)
                at = 12 + (name_size + 3) // 4 * 4
                for k in msgpack.unpackb(note[at:at + size], strict_map_key=False)["amdhsa.kernels"]:
                    out[k[".name"]] = k
    assert len(out) > 100
    return out


@pytest.mark.parametrize("kernel", ["k_head_fused", "k_head_stream", "k_proj_stream"])
def test_no_spills(kernels, kernel):
    mine = {n: k for n, k in kernels.items() if re.match(r"_ZN4soma\d+%s[IE]" % kernel, n)}
    assert mine
    spilled = {n: k[".vgpr_spill_count"] for n, k in mine.items()
               if k[".vgpr_spill_count"] or k[".private_segment_fixed_size"]}
    assert not spilled
