"""Properties of the compiled gfx950 kernels that the sources rely on, read from
the code objects of the built library.

The tiled GEMM keeps a tile's accumulators and fragments in all 256 registers of
a wave and counts its outstanding loads itself, so a value spilled to scratch
memory costs memory traffic on every tile, and inside a counted stretch it would
break the counts."""

import os
import re
import shutil
import subprocess

import pytest

from paper_2605_06206_amd import build as build_mod

LLVM = "/opt/rocm/llvm/bin"


def _tool(name):
    path = shutil.which(name, path=LLVM) or shutil.which(name)
    if path is None:
        pytest.skip(f"{name} not found")
    return path


@pytest.fixture(scope="module")
def code_objects(tmp_path_factory):
    """The gfx950 code objects of libfoe.so, one per translation unit."""
    if not os.path.exists(build_mod.LIB_PATH):
        build_mod.build()
    tmp = tmp_path_factory.mktemp("code")
    fat = str(tmp / "fatbin")
    subprocess.run([_tool("llvm-objcopy"), f"--dump-section=.hip_fatbin={fat}",
                    build_mod.LIB_PATH, str(tmp / "lib.so")], check=True)
    data = open(fat, "rb").read()
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    paths = []
    for m in re.finditer(magic, data):
        at = m.start() + len(magic)
        n = int.from_bytes(data[at:at + 8], "little")
        at += 8
        for _ in range(n):
            off, size, tlen = (int.from_bytes(data[at + 8 * i:at + 8 * i + 8], "little")
                               for i in range(3))
            triple = data[at + 24:at + 24 + tlen].decode()
            at += 24 + tlen
            if "gfx950" in triple and size:
                path = str(tmp / f"co{len(paths)}")
                with open(path, "wb") as f:
                    f.write(data[m.start() + off:m.start() + off + size])
                paths.append(path)
    assert len(paths) == len(build_mod.SOURCES)
    return paths


def _kernels(code_objects):
    """name -> fields of the kernel metadata."""
    out = {}
    for path in code_objects:
        text = subprocess.run([_tool("llvm-readelf"), "--notes", path], check=True,
                              capture_output=True, text=True).stdout
        for block in re.split(r"\n  - (?=\.\w+:)", text)[1:]:
            fields = dict(re.findall(r"^\s*(\.\w+):\s+(\S+)", block, re.M))
            if ".symbol" in fields:
                out[fields[".symbol"]] = fields
    return out


def test_no_vector_register_is_spilled(code_objects):
    kernels = _kernels(code_objects)
    assert any("ffn_fused_dma" in k for k in kernels) and len(kernels) > 40
    spilled = {k: f[".vgpr_spill_count"] for k, f in kernels.items()
               if int(f[".vgpr_spill_count"])}
    assert not spilled
    scratch = {k: f[".private_segment_fixed_size"] for k, f in kernels.items()
               if ("gemm" in k or "ffn" in k or "attn" in k)
               and int(f[".private_segment_fixed_size"])}
    assert not scratch
