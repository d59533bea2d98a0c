"""What the built kernels take of a compute unit, from the metadata of the code objects inside libcorey.so: the speeds that the
dispatch counts on rest on it, and no result shows when it changes."""
from __future__ import annotations

import os
import re
import struct

import pytest

msgpack = pytest.importorskip("msgpack")

from paper_2604_10597_amd import build


def _code_objects(lib: bytes):
    """The gfx950 code objects of the offload bundles inside a host library."""
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    at = lib.find(magic)
    while at >= 0:
        (entries,) = struct.unpack_from("<Q", lib, at + len(magic))
        pos = at + len(magic) + 8
        for _ in range(entries):
            offset, size, idlen = struct.unpack_from("<QQQ", lib, pos)
            name = lib[pos + 24:pos + 24 + idlen]
            pos += 24 + idlen
            if b"gfx950" in name and size:
                yield lib[at + offset:at + offset + size]
        at = lib.find(magic, at + len(magic))


def _kernels(obj: bytes):
    """The kernels' entries of a code object's metadata note."""
    (shoff,) = struct.unpack_from("<Q", obj, 0x28)
    shentsize, shnum = struct.unpack_from("<HH", obj, 0x3A)
    for i in range(shnum):
        kind, = struct.unpack_from("<I", obj, shoff + i * shentsize + 4)
        if kind != 7:                                           # SHT_NOTE
            continue
        pos, size = struct.unpack_from("<QQ", obj, shoff + i * shentsize + 24)
        namesz, descsz, _ = struct.unpack_from("<III", obj, pos)
        desc = pos + 12 + (namesz + 3) // 4 * 4
        yield from msgpack.unpackb(obj[desc:desc + descsz], strict_map_key=False).get("amdhsa.kernels", [])


@pytest.fixture(scope="module")
def kernels():
    if not os.path.exists(build.LIB):
        build.build_lib()
    with open(build.LIB, "rb") as f:
        lib = f.read()
    found = {k[".name"]: k for obj in _code_objects(lib) for k in _kernels(obj)}
    assert found
    return found


def _scan_kernels(kernels, storage: str):
    """Of one storage type (f: binary32, t: bf16, DF16_: binary16)."""
    out = {n: k for n, k in kernels.items() if re.match(rf"_ZN10corey_scan\d+k_scan(_any|_mix)?I{storage}L", n)}
    assert len(out) > 20
    return out


def test_binary32_staging_begins_at_the_start_of_lds(kernels):
    """The buffers that B and C are copied into are the first words of the dynamic LDS; anything static comes before them."""
    for name, k in _scan_kernels(kernels, "f").items():
        assert k[".group_segment_fixed_size"] == 0, name


def test_a_scan_kernel_has_one_body():
    """The units instantiate parts of the same templates: nothing but where k_scan_any is instantiated may depend on the unit, or one
    name has two bodies."""
    for name in sorted(os.listdir(build.CSRC)):
        if name.startswith("corey_scan"):
            with open(os.path.join(build.CSRC, name)) as f:
                text = f.read()
            used = set(re.findall(r"^#\s*(?:ifdef|ifndef|if|elif)\s+(?:!?defined\W*)?(\w+)", text, re.M))
            assert used <= {"COREY_SCAN_ANY_HERE", name.upper().replace(".", "_")}, (name, used)


@pytest.mark.parametrize("storage, steps, waves", [("f", 4, 3), ("f", 8, 2), ("f", 16, 2), ("t", 4, 3), ("t", 8, 3), ("t", 16, 3),
                                                   ("DF16_", 4, 3), ("DF16_", 8, 3), ("DF16_", 16, 3)])
def test_direct_kernels_fit_the_waves_they_are_launched_for(kernels, storage, steps, waves):
    """A SIMD's 512 registers, in blocks of 8 a wave: launches that read B and C directly go out with as many waves as these hold."""
    mine = [k for n, k in kernels.items() if re.match(rf"_ZN10corey_scan6k_scanI{storage}Li{steps}ELi\d+ELb1E", n)]
    assert mine
    for k in mine:
        assert k[".vgpr_count"] <= 512 // waves // 8 * 8, k[".name"]
