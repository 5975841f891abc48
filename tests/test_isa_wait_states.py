"""Wait states in the compiled kernels.

gfx950 does not interlock some pairs of vector instructions; the program has to
keep wait states between them.  The compiler does so for its own instructions,
but not between these and the text of an inline asm statement.  This test
disassembles the built library's gfx950 code (fall-through paths and the taken
side of every branch) and looks for pairs that stand too close:

  vector write of a scalar register -> vector read of it                 2
                                    -> lane select of readlane/writelane 4
                                    -> memory instruction reading it     5
  vector write of vcc               -> v_div_fmas                        4
  vector write of a vector register -> v_readlane / v_readfirstlane      1
                                    -> DPP read                          2
  transcendental result, or a result in part of a register -> use        1

Runs on the CPU (nothing is launched).
"""
import os
import re
import shutil
import struct
import subprocess

import pytest

from paper_1806_08815_amd import build

REG = re.compile(r"\b([sva])\[(\d+):(\d+)\]|\b([sva])(\d+)\b|\b(vcc|vcc_lo|vcc_hi)\b")
TWO_DST = re.compile(r"v_(add_co|sub_co|subrev_co|addc_co|subb_co|subbrev_co|div_scale|"
                     r"mad_u64_u32|mad_i64_i32|swap)")
TRANS = re.compile(r"v_(log|exp|rcp|rsq|sqrt|sin|cos)(_legacy|_iflag)?_f(16|32|64)")
MEMORY = ("global_", "buffer_", "flat_", "scratch_")
DEPTH = 5   # the longest distance asked for


def _objdump():
    for c in ("/opt/rocm/llvm/bin/llvm-objdump", shutil.which("llvm-objdump")):
        if c and os.path.exists(c):
            return c
    return None


def code_objects(path):
    """The gfx950 code objects bundled in a host library."""
    with open(path, "rb") as f:
        data = f.read()
    magic, p, out = b"__CLANG_OFFLOAD_BUNDLE__", 0, []
    while (p := data.find(magic, p)) >= 0:
        n, = struct.unpack_from("<Q", data, p + 24)
        q = p + 32
        for _ in range(n):
            off, size, tlen = struct.unpack_from("<QQQ", data, q)
            triple = data[q + 24:q + 24 + tlen]
            q += 24 + tlen
            if b"gfx950" in triple and size:
                out.append(data[p + off:p + off + size])
        p += len(magic)
    return out


def _regs(operand):
    out = []
    for m in REG.finditer(operand):
        if m.group(1):
            out += [(m.group(1), i) for i in range(int(m.group(2)), int(m.group(3)) + 1)]
        elif m.group(4):
            out.append((m.group(4), int(m.group(5))))
        else:
            out += [("s", r) for r in {"vcc": (106, 107), "vcc_lo": (106,),
                                       "vcc_hi": (107,)}[m.group(6)]]
    return out


class Insn:
    """What the checks need of one instruction's text."""
    seen = {}

    def __new__(cls, text):
        got = cls.seen.get(text)
        if got is None:
            got = cls.seen[text] = super().__new__(cls)
            got._decode(text)
        return got

    def _decode(self, text):
        name, _, rest = text.partition(" ")
        ops = [o.strip() for o in re.split(r",(?![^\[(]*[\])])", rest)] if rest else []
        self.text, self.name = text, name
        self.valu = name.startswith("v_")
        self.mem = name.startswith(MEMORY)
        self.wait = int(ops[0], 0) + 1 if name == "s_nop" else 1
        self.ends = name.startswith(("s_branch", "s_endpgm", "s_setpc"))
        self.branch = name.startswith(("s_branch", "s_cbranch"))
        self.dpp = "row_" in rest or "quad_perm" in rest
        self.to_lane = name.startswith(("v_readlane", "v_readfirstlane"))
        self.trans = TRANS.match(name) is not None
        self.part = "dst_sel:" in rest and "dst_sel:DWORD" not in rest
        self.fmas = name.startswith("v_div_fmas")
        self.writes, reads = set(), []
        self.select = set()
        if self.valu:
            n = 2 if TWO_DST.match(name) else 1
            self.writes = {r for o in ops[:n] for r in _regs(o)}
            reads = [r for o in ops[n:] for r in _regs(o)]
            if name.startswith(("v_fmac", "v_mac", "v_dot", "v_writelane", "v_swap")) or self.dpp \
                    or "UNUSED_PRESERVE" in rest:
                reads += self.writes
            if self.fmas or name == "v_cndmask_b32_e32":
                reads += [("s", 106), ("s", 107)]
            if name.startswith(("v_readlane", "v_writelane")):
                self.select = set(_regs(ops[2]))
        elif self.mem:
            reads = [r for o in ops for r in _regs(o)]
        self.reads = set(reads)


def _needed(first, second):
    """Wait states that `second` has to keep from `first`."""
    need = 0
    for r in first.writes & (second.reads | second.select):
        if r[0] == "s":
            need = max(need, 4 if r in second.select else 0, 5 if second.mem else 2,
                       4 if second.fmas else 0)
        elif second.valu and r in second.reads:
            need = max(need, 1 if second.to_lane else 0, 2 if second.dpp else 0,
                       1 if first.trans and not second.trans else 0, 1 if first.part else 0)
    return need


def _check(before, insns, where, bad):
    """Every instruction of `insns` against those before it (the last is nearest)."""
    window = list(before)
    for ins in insns:
        if ins.valu or ins.mem:
            states = 0
            for p in reversed(window):
                if states >= DEPTH:
                    break
                if p.valu and p.writes and _needed(p, ins) > states:
                    bad.append(f"{where}: {p.text} -> {ins.text}")
                    break
                states += p.wait
        window.append(ins)
        if len(window) > DEPTH + 3:
            window.pop(0)
        if ins.ends:
            window.clear()


def hazards(path, tmp, objdump):
    bad, count = [], 0
    for n, code in enumerate(code_objects(path)):
        elf = os.path.join(tmp, f"{n}.elf")
        with open(elf, "wb") as f:
            f.write(code)
        r = subprocess.run([objdump, "-d", "--no-show-raw-insn", elf], capture_output=True,
                           text=True, timeout=300)
        assert r.returncode == 0, r.stderr[-2000:]
        functions, name = {}, None
        for line in r.stdout.splitlines():
            if line.startswith("\t"):
                text, _, note = line.partition("//")
                addr = note.split(":", 1)[0].strip()
                if addr:   # (runs of zero bytes have none)
                    functions[name].append((int(addr, 16), " ".join(text.split()), note))
            elif line.endswith(">:"):
                name = line.split("<", 1)[1][:-2]
                functions[name] = []
        for name, body in functions.items():
            insns = [Insn(t) for _, t, _ in body]
            count += len(insns)
            _check([], insns, name, bad)
            at = {a: i for i, (a, _, _) in enumerate(body)}
            for i, ins in enumerate(insns):
                if not ins.branch:
                    continue
                m = re.search(r"\+0x([0-9a-f]+)>", body[i][2])
                to = at.get(body[0][0] + (int(m.group(1), 16) if m else 0))
                assert to is not None, (name, body[i])
                _check(insns[max(i - DEPTH, 0):i + 1], insns[to:to + DEPTH], name + " (branch)", bad)
    return bad, count


def test_no_vector_hazard_in_built_code(tmp_path):
    objdump = _objdump()
    if objdump is None:
        pytest.skip("llvm-objdump not found")
    if not os.path.exists(build.LIB):
        build.build_library()
    bad, count = hazards(build.LIB, str(tmp_path), objdump)
    assert count > 500_000        # the kernels were found
    assert not bad, (len(bad), bad[:5])


def test_the_check_sees_each_pair():
    def run(*text):
        bad = []
        _check([], [Insn(t) for t in text], "t", bad)
        return len(bad)
    lane = "v_readlane_b32 s0, v47, 9"
    use = "v_bitop3_b32 v39, v39, v40, s0 bitop3:0x96"
    assert run(lane, use) == 1 and run(lane, "s_nop 0", use) == 1 and run(lane, "s_nop 1", use) == 0
    assert run(lane, "s_nop 3", "global_load_dword v1, v2, s[0:1]") == 1
    assert run(lane, "s_nop 2", "v_readlane_b32 s4, v1, s0") == 1
    assert run(lane, "s_nop 3", "v_readlane_b32 s4, v1, s0") == 0
    assert run("v_cndmask_b32 v1, v2, v3, s[4:5]", "v_readlane_b32 s0, v1, 3") == 1
    assert run("v_add_u32_e32 v1, v2, v3", "s_nop 0",
               "v_add_u32_dpp v4, v1, v4 row_shr:1 row_mask:0xf bank_mask:0xf") == 1
    assert run("v_log_f32_e32 v1, v1", "v_add_f32_e32 v2, v1, v3") == 1
    assert run("v_log_f32_e32 v1, v1", "s_nop 0", "v_add_f32_e32 v2, v1, v3") == 0
    assert run("v_cmp_lt_u32_e32 vcc, v0, v1", "s_nop 0", "v_cndmask_b32_e32 v1, v2, v3, vcc") == 1
    assert run("v_cmp_lt_u32_e32 vcc, v0, v1", "s_branch 4", "v_cndmask_b32_e32 v1, v2, v3, vcc") == 0
