"""Registers and scratch of the built kernels, from the metadata notes of the code
objects inside the library: kernels whose comments say that nothing spills."""
import glob
import os
import re
import struct
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2408_01081_amd", "liblbm_hip.so")
READELF = "/opt/rocm/llvm/bin/llvm-readelf"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{mangled kernel name: {"scratch": B per lane, "vgpr": n, "lds": B}}"""
    if not os.path.exists(READELF):
        pytest.skip("no llvm-readelf")
    data = open(LIB, "rb").read()
    out, at = {}, data.find(MAGIC)
    d = tmp_path_factory.mktemp("co")
    while at >= 0:
        n, = struct.unpack_from("<Q", data, at + len(MAGIC))
        p = at + len(MAGIC) + 8
        for _ in range(n):
            off, size, tl = struct.unpack_from("<QQQ", data, p)
            triple = data[p + 24:p + 24 + tl]
            p += 24 + tl
            if b"gfx950" not in triple or not size:
                continue
            path = str(d / ("%d.o" % len(glob.glob(str(d / "*")))))
            with open(path, "wb") as f:
                f.write(data[at + off:at + off + size])
            text = subprocess.run([READELF, "--notes", path], capture_output=True, text=True,
                                  check=True).stdout
            for block in re.split(r"\n  - \.", text)[1:]:
                def get(k):
                    m = re.search(r"\.?\b%s:\s+(\S+)" % k, block)
                    return m and m.group(1)
                name = get("symbol")
                if name:
                    out[name.strip("'").replace(".kd", "")] = {
                        "scratch": int(get("private_segment_fixed_size")),
                        "vgpr": int(get("vgpr_count")), "lds": int(get("group_segment_fixed_size"))}
        at = data.find(MAGIC, at + 1)
    return out


def _named(kernels, name):
    found = {k: v for k, v in kernels.items() if re.search(r"\d%s(?=I|E)" % name, k)}
    assert found, name
    return found


# the surrogate's tiled kernels: two workgroups of four waves share a CU only
# within 256 registers per lane, and a reload of a spilled register waits for all
# loads in flight
@pytest.mark.parametrize("name", ["k_wgradw", "k_convw", "k_convs", "k_conv_in", "k_convt",
                                  "k_wgradt", "k_stats"])
def test_surrogate_kernels_do_not_spill(kernels, name):
    for k, v in _named(kernels, name).items():
        assert v["scratch"] == 0, (k, v)


def test_tile_kernels_are_built_for_the_largest_tile(kernels):
    # template arguments: boundary type, load, displacement, ranks, most waves.
    # Without extras the LDS is that of the 12 waves of a 24-row tile; only the
    # kernel with walls, ranks above 16 and the displacement state spills.
    tiles = _named(kernels, "k_tile")
    assert len(tiles) == 12
    for k, v in tiles.items():
        bc, load, disp, ranks = re.search(r"k_tileILi(\d)ELb(\d)ELb(\d)ELi(\d+)E", k).groups()
        if load == "0":
            assert v["lds"] <= 2 * 12 * 10 * 64 * 4 + 16, (k, v)
        if (bc, load, disp, ranks) != ("1", "1", "1", "32"):
            assert v["scratch"] == 0, (k, v)
