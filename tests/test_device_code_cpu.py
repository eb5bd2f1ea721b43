"""Properties of the compiled gfx950 kernels that the sources rely on, read from
the code objects of the built library.

The tiled GEMM keeps a tile's accumulators and fragments in all 256 registers of
a wave and counts its outstanding loads itself, so a value spilled to scratch
memory costs memory traffic on every tile, and inside a counted stretch it would
break the counts.  Its MFMAs and the LDS-DMA loads are inline assembly, around
which the compiler inserts no wait states: that none is missing is checked here,
along every path of the disassembled kernels."""

import os
import re
import shutil
import subprocess
from collections import namedtuple

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


# ---- wait states around inline assembly --------------------------------------

Instr = namedtuple("Instr", "addr op args preds")  # preds: indexes of possible predecessors
ENDS = ("s_branch", "s_endpgm", "s_setpc_b64")


def _regs(arg):
    """Registers of an operand: {('v'|'a'|'s', n)}, m0 and vcc by name."""
    arg = arg.strip().strip("-|")
    m = re.fullmatch(r"([vas])(\d+)", arg)
    if m:
        return {(m.group(1), int(m.group(2)))}
    m = re.fullmatch(r"([vas])\[(\d+):(\d+)\]", arg)
    if m:
        return {(m.group(1), i) for i in range(int(m.group(2)), int(m.group(3)) + 1)}
    return {("s", arg)} if arg in ("m0", "vcc") else set()


def parse(text):
    """Kernels of an llvm-objdump listing: name -> [Instr]."""
    out = {}
    for sect in re.split(r"\n(?=[0-9a-f]+ <)", text)[1:]:
        head = re.match(r"([0-9a-f]+) <(\S+)>:", sect)
        base, name, rows, targets = int(head.group(1), 16), head.group(2), [], {}
        for line in sect.splitlines()[1:]:
            m = re.match(r"\t(\S+)\s*(.*?)\s*// ([0-9A-F]+):[^<]*(?:<[^>+]*(?:\+0x([0-9a-f]+))?>)?", line)
            if not m:
                continue
            op, args, addr, off = m.groups()
            if "branch" in op:
                targets.setdefault(base + int(off or "0", 16), []).append(len(rows))
            rows.append((int(addr, 16), op, [a for a in args.split(",") if a]))
        out[name] = [
            Instr(a, op, args, targets.get(a, []) +
                  ([i - 1] if i and rows[i - 1][1] not in ENDS else []))
            for i, (a, op, args) in enumerate(rows)]
    return out


def _before(code, at, states):
    """Instructions that can run within `states` wait states before code[at]."""
    seen, todo = {}, [(p, 0) for p in code[at].preds]
    while todo:
        i, used = todo.pop()
        if used >= states or seen.get(i, states) <= used:
            continue
        seen[i] = used
        c = code[i]
        step = int(c.args[0], 0) + 1 if c.op == "s_nop" else 1
        if c.op != "s_nop":
            yield c
        todo += [(p, used + step) for p in c.preds]


def _is_valu(c):
    return c.op.startswith("v_") and not c.op.startswith("v_mfma")


def _writes(c):
    dst = _regs(c.args[0]) if c.args else set()
    if "swap" in c.op or "_co_" in c.op or "div_scale" in c.op:
        dst |= _regs(c.args[1])
    return dst


def mfma_faults(code):
    """MFMA operands written by a vector instruction less than two wait states
    before, and results touched by another kind of instruction less than 19 after
    (the largest number for any MFMA)."""
    bad = []
    for i, c in enumerate(code):
        if c.op.startswith("v_mfma"):
            src = set().union(*(_regs(a) for a in c.args[1:]))
            bad += [(hex(c.addr), p.op) for p in _before(code, i, 2)
                    if _is_valu(p) and _writes(p) & src]
        elif c.op.startswith(("v_", "ds_", "global_", "buffer_", "scratch_")):
            used = set().union(*(_regs(a) for a in c.args), set())
            acc = {r for r in used if r[0] == "a"}
            if acc:
                bad += [(hex(c.addr), c.op) for p in _before(code, i, 19)
                        if p.op.startswith("v_mfma") and _writes(p) & acc]
    return bad


def dma_faults(code):
    """LDS-DMA loads whose resource a vector instruction wrote less than five wait
    states before, or whose M0 is not set by the scalar add one wait state before;
    any other use of M0."""
    bad = []
    for i, c in enumerate(code):
        if c.op.startswith("buffer_load") and c.args[-1].rstrip().endswith("lds"):
            rsrc = _regs(c.args[1])
            bad += [(hex(c.addr), p.op) for p in _before(code, i, 5)
                    if _is_valu(p) and _writes(p) & rsrc]
            if not (i >= 2 and code[i - 1].op == "s_nop" and c.preds == [i - 1] and
                    code[i - 1].preds == [i - 2] and code[i - 2].op == "s_add_u32" and
                    code[i - 2].args[0] == "m0"):
                bad.append((hex(c.addr), "m0"))
        elif any("m0" == a.strip() for a in c.args):
            nxt = code[i + 2] if i + 2 < len(code) else None
            if not (c.op == "s_add_u32" and nxt and nxt.op.startswith("buffer_load")):
                bad.append((hex(c.addr), c.op))
    return bad


@pytest.fixture(scope="module")
def kernels(code_objects):
    out = {}
    for path in code_objects:
        out.update(parse(subprocess.run([_tool("llvm-objdump"), "-d", "--no-show-raw-insn", path],
                                        check=True, capture_output=True, text=True).stdout))
    return out


def test_inline_mfmas_have_their_wait_states(kernels):
    tiled = {k: c for k, c in kernels.items() if "grouped_gemm_dma" in k or "ffn_fused_dma" in k}
    assert len(tiled) >= 10
    for name, code in tiled.items():
        assert sum(c.op.startswith("v_mfma") for c in code) >= 32, name
        assert not mfma_faults(code), name


def test_lds_dma_loads_have_their_wait_states(kernels):
    n = 0
    for name, code in kernels.items():
        n += sum(c.op.startswith("buffer_load") and c.args[-1].endswith("lds") for c in code)
        assert not dma_faults(code), name
    assert n > 100


def _loops(code):
    """Bodies of the innermost loops: from a branch's target to the branch."""
    found = []
    for i, c in enumerate(code):
        found += [(i, p) for p in c.preds if p > i]
    inner = [(a, b) for a, b in found
             if not any(a <= x and y <= b and (x, y) != (a, b) for x, y in found)]
    return [code[a:b + 1] for a, b in inner]


def test_waves_without_rows_run_no_mfmas(kernels):
    """The 256-row kernels have a K loop with loads and barriers alone, for waves
    none of whose tile rows exist, beside the full one and the half one."""
    tiled = {k: c for k, c in kernels.items()
             if "ffn_fused_dma" in k or ("grouped_gemm_dma" in k and "Li256E" in k)}
    assert len(tiled) >= 3
    for name, code in tiled.items():
        loops = [[c.op for c in body] for body in _loops(code)]
        loops = [ops for ops in loops if "s_barrier" in ops and
                 any(op.startswith("buffer_load_dwordx4") for op in ops)]
        mfmas = sorted({sum(op.startswith("v_mfma") for op in ops) for ops in loops})
        assert len(mfmas) == 3 and mfmas[0] == 0 and mfmas[2] == 2 * mfmas[1], (name, mfmas)


LISTING = """
x:	file format elf64-amdgpu

0000000000000100 <k>:
\tv_mov_b32_e32 v4, v9                                       // 000000000100: 00
\ts_branch 1                                                 // 000000000104: 00 <k+0xc>
\tv_mov_b32_e32 v5, v9                                       // 000000000108: 00
\t{mid}                                                      // 00000000010C: 00
\tv_mfma_f32_16x16x32_bf16 a[0:3], v[4:7], v[8:11], a[0:3]   // 000000000110: 00
\ts_nop {nop}                                                // 000000000114: 00
\tv_accvgpr_read_b32 v1, a2                                  // 000000000118: 00
\tv_readfirstlane_b32 s9, v1                                 // 00000000011C: 00
\ts_nop 1                                                    // 000000000120: 00
\ts_add_u32 m0, s3, 0x400                                    // 000000000124: 00
\ts_nop {nop2}                                               // 000000000128: 00
\tbuffer_load_dwordx4 v2, s[8:11], 0 offen lds               // 00000000012C: 00
\ts_endpgm                                                   // 000000000130: 00
"""


def test_scanner_sees_missing_wait_states():
    """The checks above on a listing of their own: with too few wait states on one
    path (through the branch, or straight on) and with enough on both."""
    def faults(**kw):
        code = parse(LISTING.format(**kw))["k"]
        return [op for _, op in mfma_faults(code)], [op for _, op in dma_faults(code)]

    assert faults(mid="s_nop 1", nop=15, nop2=3) == (["v_accvgpr_read_b32"], [])
    assert faults(mid="s_nop 1", nop=18, nop2=1) == ([], [])
    assert faults(mid="s_nop 1", nop=18, nop2=0) == ([], ["v_readfirstlane_b32"])
    assert faults(mid="s_mov_b32 s1, s2", nop=18, nop2=1) == (["v_mov_b32_e32"], [])
    assert faults(mid="v_mov_b32_e32 v11, v9", nop=18, nop2=1) == (
        ["v_mov_b32_e32", "v_mov_b32_e32"], [])
    assert faults(mid="s_mov_b32 m0, s2", nop=18, nop2=1)[1] == ["s_mov_b32"]
