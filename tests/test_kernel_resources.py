"""What the compiler made of the kernels, from the built library's own metadata (no GPU): the
work-groups that a kernel's launch bounds ask for fit a compute unit."""
import os
import re
import struct

import pytest

from paper_2505_24504_amd import jfmg

msgpack = pytest.importorskip("msgpack")

LDS_BYTES = 160 * 1024   # of a compute unit, shared by its work-groups
VGPRS = 512              # of a SIMD's lane, shared by its waves


def code_objects(data):
    """The gfx950 code objects of a library: the entries of its offload bundles."""
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    at = data.find(magic)
    while at >= 0:
        n = struct.unpack_from("<Q", data, at + 24)[0]
        pos = at + 32
        for _ in range(n):
            off, size, tl = struct.unpack_from("<QQQ", data, pos)
            if b"gfx950" in data[pos + 24:pos + 24 + tl]:
                yield data[at + off:at + off + size]
            pos += 24 + tl
        at = data.find(magic, at + 24)


def kernels(elf):
    """Metadata records of a code object's kernels (the AMDGPU note's MessagePack)."""
    shoff, = struct.unpack_from("<Q", elf, 40)
    shentsize, shnum = struct.unpack_from("<HH", elf, 58)
    for i in range(shnum):
        sh = shoff + i * shentsize
        kind, = struct.unpack_from("<I", elf, sh + 4)
        off, size = struct.unpack_from("<QQ", elf, sh + 24)
        if kind != 7:   # SHT_NOTE
            continue
        end = off + size
        while off < end:
            nl, dl, _ = struct.unpack_from("<III", elf, off)
            name, desc = off + 12, off + 12 + (nl + 3) // 4 * 4
            if elf[name:name + nl].rstrip(b"\0") == b"AMDGPU":
                yield from msgpack.unpackb(elf[desc:desc + dl])["amdhsa.kernels"]
            off = desc + (dl + 3) // 4 * 4


@pytest.fixture(scope="module")
def records():
    if not os.path.exists(jfmg.LIB_PATH):
        from paper_2505_24504_amd import build
        build.build()
    with open(jfmg.LIB_PATH, "rb") as fh:
        data = fh.read()
    out = {k[".name"]: k for o in code_objects(data) for k in kernels(o)}
    assert len(out) > 300
    return out


def test_fv_tile_kernels_fit_their_launch_bounds(records):
    """fv_tile_kernel<T, TX, TZ, threads, waves per SIMD, ...>: as many work-groups fit a
    compute unit's LDS and registers as give each of its four SIMDs that many waves."""
    n = 0
    for name, k in records.items():
        m = re.match(r"_ZN4jfmg14fv_tile_kernelI[df]Li\d+ELi\d+ELi(\d+)ELi(\d+)E", name)
        if not m:
            continue
        threads, waves = int(m[1]), int(m[2])
        groups = max(1, 4 * waves // (threads // 64))
        lds, vgprs = k[".group_segment_fixed_size"], k[".vgpr_count"]
        assert groups * lds <= LDS_BYTES, (name, lds)
        assert vgprs <= VGPRS // waves and k[".private_segment_fixed_size"] == 0, (name, vgprs)
        n += 1
    assert n >= 200   # 2 types, 6 shapes, 6 modes, single, lock-step and ragged
