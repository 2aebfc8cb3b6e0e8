"""Checks the gfx950 code of built objects: no instruction touches a register that an LDS read in flight will write.

The tile kernels issue their LDS reads in one asm statement and wait for them in another, so that reads, copies and MFMAs
overlap.  For the compiler such a read's output is written at once: a copy of it (to another register, an accumulation
register or scratch memory) placed before the wait would take a stale value, and the register, free from there on, could
hold an address when the data arrives.  Nothing in the language rules that out, so build.py looks at the code that came out
and fails where it happened; and where a kernel with private rings (spmm_rings.hip) spills or uses accumulation registers.

    python -m paper_2407_20496_amd.lds_reads OBJECT...

How it looks: the instructions of a function as basic blocks; along every path the LDS operations that may be outstanding,
newest first, each with the registers it will write.  LDS operations finish in order, so `s_waitcnt lgkmcnt(n)` leaves
the n newest at most; scalar loads count there too, which only means that fewer than n are left.
"""
from __future__ import annotations

import os
import re
import subprocess
import sys
import tempfile

LLVM = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin")
TARGET = "hip-amdgcn-amd-amdhsa--gfx950"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"
KEEP = 16       # outstanding operations told apart (the hardware's counter reaches 15); older ones are lumped together

_REGS = re.compile(r"\b([va])(?:(\d+)\b|\[(\d+):(\d+)\])")
_WAIT = re.compile(r"lgkmcnt\((\d+)\)")
_LINE = re.compile(r"^\s+(\S+)(?:\s+(.*?))?\s*// ([0-9A-Fa-f]+):[^<]*(?:<(.+?)(?:\+0x([0-9a-fA-F]+))?>)?\s*$")
_LABEL = re.compile(r"^([0-9a-fA-F]+) <(.+)>:$")


def _run(*cmd: str) -> str:
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError(f"{os.path.basename(cmd[0])} failed: {res.stderr.strip()}")
    return res.stdout


def code_objects(obj: str, directory: str):
    """The gfx950 code objects inside a host object or shared library that hipcc wrote (a library holds one of each source)."""
    section, bundle, code = (os.path.join(directory, f) for f in ("section", "bundle", "code"))
    _run(os.path.join(LLVM, "llvm-objcopy"), "--dump-section", ".hip_fatbin=" + section, obj, os.path.join(directory, "copy"))
    with open(section, "rb") as f:
        bundles = f.read().split(MAGIC)[1:]
    for body in bundles:
        with open(bundle, "wb") as f:
            f.write(MAGIC + body)
        _run(os.path.join(LLVM, "clang-offload-bundler"), "--unbundle", "--type=o", "--targets=" + TARGET,
             "--input=" + bundle, "--output=" + code)
        yield code


def _registers(text: str) -> set:
    out = set()
    for kind, one, first, last in _REGS.findall(text):
        if one:
            out.add(kind + one)
        else:
            out.update(kind + str(r) for r in range(int(first), int(last) + 1))
    return out


def functions(disassembly: str):
    """(name, [(address, mnemonic, operands, branch target or None)]) of every function of `llvm-objdump -d`."""
    name, code, start = None, [], 0
    for line in disassembly.splitlines():
        label = _LABEL.match(line)
        if label:
            if name and code:
                yield name, code
            name, code, start = label[2], [], int(label[1], 16)
            continue
        ins = _LINE.match(line)
        if ins and name:
            target = start + int(ins[5] or "0", 16) if ins[4] == name else None
            code.append((int(ins[3], 16), ins[1], ins[2] or "", target))
    if name and code:
        yield name, code


def _step(state: tuple, mnemonic: str, operands: str):
    """State after one instruction, and the registers in flight that it touches."""
    touched = set()
    if state and not mnemonic.startswith("s_"):
        flying = set().union(*state)
        if flying:
            touched = _registers(operands) & flying
    if mnemonic == "s_waitcnt":
        left = _WAIT.search(operands)
        if left:
            state = state[:int(left[1])]
    elif mnemonic.startswith("ds_") and mnemonic != "ds_nop":
        reads = re.match(r"ds_(read|load|bpermute|permute|swizzle|.*_rtn)", mnemonic) is not None
        new = frozenset(_registers(operands.split(",")[0])) if reads else frozenset()
        state = (new,) + state
        if len(state) > KEEP:
            state = state[:KEEP - 1] + (frozenset().union(*state[KEEP - 1:]),)
    return state, touched


def _join(a: tuple, b: tuple) -> tuple:
    if len(a) < len(b):
        a, b = b, a
    return tuple(x | b[i] if i < len(b) else x for i, x in enumerate(a))


def violations(disassembly: str) -> list:
    """Texts, one for each instruction that touches a register an LDS read in flight will write."""
    found = []
    for name, code in functions(disassembly):
        if not any(m.startswith("ds_") for _, m, _, _ in code):
            continue
        index = {address: i for i, (address, _, _, _) in enumerate(code)}
        starts = {0} | {index[t] for _, _, _, t in code if t is not None}
        starts |= {i + 1 for i, (_, m, _, _) in enumerate(code) if m.startswith(("s_branch", "s_cbranch", "s_endpgm"))}
        starts = sorted(s for s in starts if s < len(code))
        end_of = {s: (starts[k + 1] if k + 1 < len(starts) else len(code)) for k, s in enumerate(starts)}
        entry, todo, bad = {0: ()}, [0], {}
        while todo:
            block = todo.pop()
            state = entry[block]
            for i in range(block, end_of[block]):
                _, mnemonic, operands, _ = code[i]
                state, touched = _step(state, mnemonic, operands)
                if touched:
                    bad[i] = touched
            _, last, _, target = code[end_of[block] - 1]
            following = [] if last in ("s_branch", "s_endpgm") else [end_of[block]]
            if target is not None:
                following.append(index[target])
            for f in following:
                if f >= len(code):
                    continue
                joined = _join(entry[f], state) if f in entry else state
                if entry.get(f) != joined:
                    entry[f] = joined
                    todo.append(f)
        for i in sorted(bad):
            found.append(f"{name}: {code[i][0]:x}: {code[i][1]} {code[i][2]} ({', '.join(sorted(bad[i]))} in flight)")
    return found


def resources(notes: str) -> dict:
    """{kernel: (accumulation registers, spilled vector registers, bytes of scratch memory)} of `llvm-readelf --notes`."""
    out = {}
    for entry in re.split(r"\n\s*- \.agpr_count:", notes)[1:]:
        field = lambda key: re.search(r"\n\s*\." + key + r":\s*(\S+)", entry)[1]
        out[field("name")] = (int(entry.split(None, 1)[0]), int(field("vgpr_spill_count")), int(field("private_segment_fixed_size")))
    return out


def disassembly(code: str) -> str:
    return _run(os.path.join(LLVM, "llvm-objdump"), "-d", "--no-show-raw-insn", code)


def check(obj: str) -> list:
    """Texts, one for each fault of the built object or library."""
    found = []
    with tempfile.TemporaryDirectory() as directory:
        for code in code_objects(obj, directory):
            found += violations(disassembly(code))
            for name, used in resources(_run(os.path.join(LLVM, "llvm-readelf"), "--notes", code)).items():
                if "RingParams" in name and any(used):     # spmm_rings.hip: fragments fill the registers, none may go elsewhere
                    found.append("%s: %d accumulation registers, %d spilled, %d bytes of scratch memory" % (name, *used))
    return found


if __name__ == "__main__":
    faults = [f"{o}: {f}" for o in sys.argv[1:] for f in check(o)]
    print("\n".join(faults[:40]))
    sys.exit(1 if faults else 0)
