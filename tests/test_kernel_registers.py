"""Register budgets that the launches of libcrk.so count on, read from the
metadata of its gfx950 code objects: a SIMD has 512 registers per lane, so a
kernel with at most 256 runs two wavefronts per SIMD, 168 three, 128 four."""
import struct
import subprocess

import pytest

msgpack = pytest.importorskip("msgpack")

from paper_2604_02125_amd import crk


def _notes(elf):
    """kernel metadata of one code object (the AMDGPU note is a msgpack map)"""
    shoff, = struct.unpack_from("<Q", elf, 40)
    size, count = struct.unpack_from("<HH", elf, 58)
    for k in range(count):
        kind, = struct.unpack_from("<I", elf, shoff + k * size + 4)
        off, = struct.unpack_from("<Q", elf, shoff + k * size + 24)
        if kind == 7:                                  # SHT_NOTE
            name, desc, typ = struct.unpack_from("<III", elf, off)
            if typ == 32:                              # NT_AMDGPU_METADATA
                d = off + 12 + (name + 3) // 4 * 4
                yield from msgpack.unpackb(elf[d:d + desc])["amdhsa.kernels"]


@pytest.fixture(scope="module")
def kernels():
    with open(crk.LIB_PATH, "rb") as fh:
        blob = fh.read()
    magic, found, i = b"__CLANG_OFFLOAD_BUNDLE__", {}, 0
    while (i := blob.find(magic, i)) >= 0:
        n, p = struct.unpack_from("<Q", blob, i + 24)[0], i + 32
        for _ in range(n if n < 16 else 0):
            off, size, length = struct.unpack_from("<QQQ", blob, p)
            if b"gfx950" in blob[p + 24:p + 24 + length]:
                for m in _notes(blob[i + off:i + off + size]):
                    found[m[".name"]] = m
            p += 24 + length
        i += len(magic)
    names = subprocess.run(["c++filt"], input="\n".join(found), capture_output=True, text=True, check=True).stdout.split("\n")
    out = {}
    for m, name in zip(found.values(), names):
        out[name.split("(")[0].replace("void ", "").replace("crk::", "")] = m
    assert len(out) > 1000
    return out


@pytest.mark.parametrize("N", [2, 3])
@pytest.mark.parametrize("flux", [0, 3])
def test_mhd_rkfr_stage_runs_two_wavefronts(kernels, N, flux):
    """GLM-MHD stages of degrees 2 and 3 in FP64 as large meshes launch them
    (one wavefront costs 10 to 20 %): the form that loads late, where there is
    one."""
    name = f"k_rkfr_stage<double, 1, 2, {N}, {flux}"
    forms = [m for k, m in kernels.items() if k in (name + ">", name + ", false>")]
    m, = forms or [kernels[name + ", true>"]]
    assert m[".vgpr_count"] <= 256 and m[".vgpr_spill_count"] == 0
