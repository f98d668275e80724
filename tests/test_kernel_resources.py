"""Registers of the kernels that carry a transform of any length, read from the
built library's own code objects (no GPU needed): a SIMD holds 512 per lane, so a
kernel with more than 256 runs one wave per SIMD, one with more than 168 two."""
import os
import re
import struct

import msgpack
import pytest

import paper_2002_01392_amd

LIB = os.path.join(os.path.dirname(paper_2002_01392_amd.__file__), "libfcns.so")
pytestmark = pytest.mark.skipif(not os.path.exists(LIB), reason="libfcns.so not built")


def _code_objects(data):
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    at = data.find(magic)
    while at >= 0:
        n, p = struct.unpack_from("<Q", data, at + 24)[0], at + 32
        for _ in range(n):
            off, size, idlen = struct.unpack_from("<QQQ", data, p)
            if b"gfx950" in data[p + 24:p + 24 + idlen]:
                yield data[at + off:at + off + size]
            p += 24 + idlen
        at = data.find(magic, at + 1)


def _kernels(elf):
    shoff, = struct.unpack_from("<Q", elf, 40)
    shentsize, shnum = struct.unpack_from("<HH", elf, 58)
    for i in range(shnum):
        h = shoff + i * shentsize
        kind, = struct.unpack_from("<I", elf, h + 4)
        if kind != 7:   # SHT_NOTE
            continue
        p, size = struct.unpack_from("<QQ", elf, h + 24)
        namesz, descsz, _ = struct.unpack_from("<III", elf, p)
        desc = p + 12 + (namesz + 3) // 4 * 4
        meta = msgpack.unpackb(elf[desc:desc + descsz], strict_map_key=False)
        for k in meta["amdhsa.kernels"]:
            yield k[".name"], (k[".vgpr_count"], k[".max_flat_workgroup_size"])


@pytest.fixture(scope="module")
def registers():
    with open(LIB, "rb") as fh:
        data = fh.read()
    out = {n: v for elf in _code_objects(data) for n, v in _kernels(elf)}
    assert len(out) > 100
    return out


@pytest.mark.parametrize("kernel,least", [
    ("k_x_nl(3)?Id.*", 2),                              # x pass with products
    (r"k_yId.*DynPlan.*Li[4689]ELb[01]ELi[48]E.*", 2),  # y transforms of up to 512 points
    ("k_z_backId.*DynPlan.*", 2),                       # z back transforms
    ("k_z_(back|stageA)Id.*DynPlan.*Li4E.*", 3),        # N' <= 128
    ("k_z_passI.*SPlan.*ELi[2-5]ELb0E.*", 3),            # compiled plans of N' <= 160
    (r"k_z_stageBId.*DynPlanIL[bi]\dEEELi0E.*", 3),
])
def test_waves_per_simd(registers, kernel, least):
    got = {n: v for n, v in registers.items() if re.search(r"4fcns\d+" + kernel, n)}
    assert got, kernel
    most = {2: 256, 3: 168}[least]
    assert not {n: v for n, (v, _) in got.items() if v > most}


@pytest.mark.parametrize("lines,threads", [(8, 256), (4, 512)])
def test_threads_of_the_x_tiles(registers, lines, threads):
    # rows above 256 points have half the lines, and twice the threads, per tile
    got = {n: t for n, (_, t) in registers.items()
           if re.search(rf"4fcns\d+k_x_(r2c|c2r)ILi{lines}E", n)}
    assert len(got) == 6 and set(got.values()) == {threads}
