"""A vector-memory instruction must not read a scalar register within five wait states of the vector instruction that wrote it
(v_readfirstlane, a comparison's mask, ...).  The compiler keeps that distance for its own instructions, not for those in inline assembly, which
is how the direct global->LDS loads are written.  The built kernels are disassembled and every such read is followed back over all ways to it."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2502_05431_amd import build as BUILD

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
NEED = 5
TWO_RESULTS = ("v_add_co", "v_sub_co", "v_subrev_co", "v_addc", "v_subb", "v_div_scale", "v_mad_u64", "v_mad_i64")


def _scalars(text):
    """The scalar registers that an operand names."""
    m = re.fullmatch(r"s\[(\d+):(\d+)\]|s(\d+)|(vcc(?:_lo|_hi)?)", text)
    if not m:
        return frozenset()
    if m[4]:
        return frozenset({"vcc": (106, 107), "vcc_lo": (106,), "vcc_hi": (107,)}[m[4]])
    return frozenset(range(int(m[1]), int(m[2]) + 1) if m[1] else (int(m[3]),))


def _operands(args):
    return [t for t in re.split(r"[,\s]+", args) if t]


def _kernels(listing):
    """(name, address, [(opcode, operands, address, target or None)])"""
    out = []
    for line in listing.splitlines():
        head = re.match(r"([0-9a-f]+) <(.*)>:", line)
        if head:
            out.append((head[2], int(head[1], 16), []))
            continue
        m = re.match(r"\t(\S+)\s*(.*?)\s*// ([0-9A-F]+):.*?(?:<[^<>]*?(?:\+0x([0-9a-f]+))?>)?$", line)
        if m and out:
            branch = m[1].startswith(("s_branch", "s_cbranch"))
            out[-1][2].append((m[1], _operands(m[2]), int(m[3], 16), out[-1][1] + int(m[4] or "0", 16) if branch else None))
    return out


def too_close(listing):
    """How many vector-memory instructions read scalar registers, and those that do so too early."""
    reads, found = 0, []
    for name, _, code in _kernels(listing):
        at = {c[2]: i for i, c in enumerate(code)}
        before = [[] for _ in code]
        for i, (op, _, _, target) in enumerate(code):
            if i + 1 < len(code) and op not in ("s_branch", "s_endpgm"):
                before[i + 1].append(i)
            if target is not None:
                before[at[target]].append(i)
        for i, (op, args, addr, _) in enumerate(code):
            regs = frozenset().union(*map(_scalars, args)) if re.match(r"(global|buffer|scratch|flat)_", op) else None
            if not regs:
                continue
            reads += 1
            todo, seen = [(p, 0, regs) for p in before[i]], set()
            while todo:
                p, waited, regs = todo.pop()
                if waited >= NEED or not regs or (p, waited, regs) in seen:
                    continue
                seen.add((p, waited, regs))
                o, a, _, _ = code[p]
                wrote = frozenset().union(*map(_scalars, a[:2] if o.startswith(TWO_RESULTS) else a[:1]))
                if o.startswith("v_") and wrote & regs:
                    found.append("%s: %s %s at %x, %d wait states behind %s %s" % (name, op, " ".join(args), addr, waited, o, " ".join(a)))
                    break
                if o.startswith(("v_", "s_")) and not o.startswith(("s_cmp", "s_bitcmp", "s_nop")):
                    regs = regs - wrote                       # (written anew behind whatever wrote it before)
                step = int(a[0], 0) + 1 if o == "s_nop" else 1
                todo += [(q, waited + step, regs) for q in before[p]]
    return reads, found


def _listing(obj, tmp_path):
    copy = str(tmp_path / "o")
    shutil.copy(obj, copy)
    subprocess.run([OBJDUMP, "--offloading", copy], check=True, capture_output=True, cwd=tmp_path)
    code = [f for f in os.listdir(tmp_path) if "gfx950" in f]
    return subprocess.run([OBJDUMP, "-d", str(tmp_path / code[0])], check=True, capture_output=True, text=True).stdout


@pytest.mark.parametrize("source, loads", [("ape_encode_walk.hip", 16), ("ape_tile_mfma.hip", 900), ("ape_flash_mfma.hip", 1000), ("ape_generic.hip", 1),
                                           ("ape_probe.hip", 1)])
def test_distance(source, loads, tmp_path):
    obj = os.path.join(os.path.dirname(BUILD.RESOURCES), source + ".o")
    files = BUILD.sources() + BUILD.probe_sources()
    if not os.path.exists(obj) or os.path.getmtime(obj) < max(os.path.getmtime(s) for s in files):
        BUILD.build(verbose=False)
    reads, found = too_close(_listing(obj, tmp_path))
    assert reads >= loads and not found, "%d of %d\n%s" % (len(found), reads, "\n".join(found[:10]))


def test_what_counts():
    """Straight code, an s_nop, a write in between, and a way around the write through a branch."""
    text = "0000000000000100 <k>:\n" + "\n".join("\t%s // %012X: 0%s" % (code, 0x100 + 4 * i, tail) for i, (code, tail) in enumerate([
        ("v_readfirstlane_b32 s0, v4", ""), ("s_mov_b32 m0, s5", ""), ("%s", ""), ("global_load_lds_dwordx4 v9, s[0:1]", ""), ("s_endpgm", "")]))
    assert len(too_close(text % "s_nop 0")[1]) == 1 and len(too_close(text % "s_nop 2")[1]) == 1
    assert too_close(text % "s_nop 3") == (1, []) and too_close(text % "s_mov_b64 s[0:1], s[8:9]") == (1, [])
    assert len(too_close(text % "s_mov_b32 s1, s9")[1]) == 1
    around = (text % "s_mov_b64 s[0:1], s[8:9]").replace("s_mov_b32 m0, s5 // 000000000104: 0", "s_cbranch_scc1 1 // 000000000104: 0 <k+0xc>")
    assert len(too_close(around)[1]) == 1
