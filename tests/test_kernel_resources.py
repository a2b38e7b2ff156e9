"""Registers and spills of the built kernels, from the library's own code
objects: a rarely taken branch sets the registers of its whole kernel, and
with them how many waves a compute unit holds."""
import os
import re
import shutil
import struct
import subprocess

import pytest

from paper_2010_02164_amd import _native

READELF = next((p for p in ("/opt/rocm/llvm/bin/llvm-readelf", shutil.which("llvm-readelf") or "") if os.path.exists(p)),
               None)
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _code_objects(lib):
    """The gfx950 code objects embedded in the library."""
    at = lib.find(MAGIC)
    while at >= 0:
        n, = struct.unpack_from("<Q", lib, at + len(MAGIC))
        p = at + len(MAGIC) + 8
        for _ in range(n):
            off, size, length = struct.unpack_from("<QQQ", lib, p)
            name = lib[p + 24:p + 24 + length]
            p += 24 + length
            if b"gfx950" in name and size:
                yield lib[at + off:at + off + size]
        at = lib.find(MAGIC, at + len(MAGIC))


@pytest.fixture(scope="module")
def kernels(native_lib, tmp_path_factory):
    """Kernel name -> (VGPRs with AGPRs, spilled VGPRs)."""
    if READELF is None:
        pytest.skip("no llvm-readelf")
    with open(_native.LIB_PATH, "rb") as f:
        lib = f.read()
    out = {}
    for i, obj in enumerate(_code_objects(lib)):
        path = tmp_path_factory.mktemp("co") / f"{i}.o"
        path.write_bytes(obj)
        notes = subprocess.run([READELF, "--notes", str(path)], capture_output=True, text=True, check=True).stdout
        for block in notes.split("  - .agpr_count:")[1:]:
            def field(key):
                return re.search(rf"\.{key}: +(\S+)", block).group(1)
            out[field("name")] = (int(field("vgpr_count")), int(field("vgpr_spill_count")))
    assert any("k_beam" in k for k in out) and any("k_proj" in k for k in out)
    return out


def test_beam_update_registers(kernels):
    """Two 8-wave beams per compute unit (128 registers a lane; 168, three waves
    per SIMD, for the row merge by itself): the recomputation of saturated tiles
    must not set the kernels' registers, nor be there where full tile lists rule
    it out."""
    beam = {k: v for k, v in kernels.items() if "k_beam" in k or "k_rowmerge" in k}
    assert len(beam) >= 10
    for name, (vgprs, spills) in beam.items():
        assert vgprs <= (168 if "k_rowmerge" in name else 128) and spills == 0, (name, vgprs, spills)


def test_projection_registers(kernels):
    """Two 4-wave workgroups per compute unit (256 registers a lane), nothing
    spilled by the epilogue's longest key lists."""
    proj = {k: v for k, v in kernels.items() if "k_proj" in k or "k_kv_append" in k}
    assert len(proj) == 7
    for name, (vgprs, spills) in proj.items():
        assert vgprs <= 256 and spills == 0, (name, vgprs, spills)
