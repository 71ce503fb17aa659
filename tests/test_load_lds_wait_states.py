"""The loads from memory straight into LDS are written in inline asm, where the compiler inserts no wait states: in the built library none of
them may read an SGPR that a vector instruction wrote fewer than five wait states earlier (CDNA: "VALU writes SGPR", then "VMEM reads that
SGPR": 5 wait states, no interlock), or follow at once a scalar instruction that wrote m0, the address in LDS (1 wait
state).  Reads the AMD assembly of the library built here."""
import os
import re
import struct
import subprocess

import pytest

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
NEEDED = 5


def _code_objects(path):
    data, magic, at = open(path, "rb").read(), b"__CLANG_OFFLOAD_BUNDLE__", 0
    while (at := data.find(magic, at)) >= 0:
        (entries,) = struct.unpack_from("<Q", data, at + 24)
        pos = at + 32
        for _ in range(entries):
            offset, size, length = struct.unpack_from("<QQQ", data, pos)
            name = data[pos + 24:pos + 24 + length]
            pos += 24 + length
            if b"gfx950" in name and size:
                yield data[at + offset:at + offset + size]
        at += len(magic)


def _sgprs(text):
    """The numbers of the SGPRs an operand list names."""
    regs = set(int(r) for r in re.findall(r"\bs(\d+)\b", text))
    for a, b in re.findall(r"\bs\[(\d+):(\d+)\]", text):
        regs.update(range(int(a), int(b) + 1))
    return regs


def hazards(lines):
    """(kernel, load, wait states, writer) of every load into LDS that comes too early, and the number of such loads.  An s_waitcnt that has
    nothing to wait for is not counted as a wait state."""
    found, loads, kernel, past = [], 0, "", []
    for line in lines:
        if (m := re.match(r"[0-9a-f]+ <(.+)>:", line)):
            kernel, past = m[1], []
            continue
        text = line.split("//")[0].strip()
        if not text or not re.match(r"[a-z]", text):
            continue
        op, _, args = text.partition(" ")
        if op.startswith("global_load_lds"):
            loads += 1
            before = [x for x in past if x[0] != "s_waitcnt"][-1:]
            if before and before[0][0].startswith("s_") and re.match(r"m0\b", before[0][1]):
                found.append((kernel, text, 0, "{} {}".format(*before[0])))
            base, waited = _sgprs(args), 0
            for pop, pargs in reversed(past):
                if waited >= NEEDED:
                    break
                dst = pargs.split(",")[0]
                if pop.startswith("v_") and _sgprs(dst) & base:
                    found.append((kernel, text, waited, f"{pop} {pargs}"))
                    break
                waited += int(pargs, 0) + 1 if pop == "s_nop" else 0 if pop == "s_waitcnt" else 1
        past.append((op, args))
        del past[:-16]
    return found, loads


def test_the_rule_on_short_sequences():
    head = ["0000 <k>:"]
    early = ["v_readfirstlane_b32 s59, v9", "v_readfirstlane_b32 s58, v8", "s_mov_b32 m0, s3", "s_waitcnt lgkmcnt(0)"]
    load = ["global_load_lds_dwordx4 v1, s[58:59]"]
    assert hazards(head + early + load)[0][-1][2] == 1
    assert not hazards(head + early + ["s_nop 3"] + load)[0]
    assert hazards(head + early + ["s_nop 2"] + load)[0]
    assert not hazards(head + early + ["s_mov_b64 s[4:5], s[58:59]", "global_load_lds_dwordx4 v1, s[4:5]"])[0]
    assert hazards(head + ["v_cmp_eq_u32_e64 s[58:59], v0, v1"] + load)[0]
    assert hazards(head + ["s_mov_b32 m0, s3", "s_waitcnt lgkmcnt(0)"] + load)[0]
    assert not hazards(head + ["s_mov_b32 m0, s3", "s_mov_b64 s[58:59], s[4:5]", "s_waitcnt lgkmcnt(0)"] + load)[0]


def test_loads_into_lds_wait_for_their_address(tmp_path):
    from paper_2512_16615_amd import build, llsa
    if not os.path.exists(llsa.LIB_PATH):
        build.build(verbose=False)
    found, loads = [], 0
    for i, code in enumerate(_code_objects(llsa.LIB_PATH)):
        obj = tmp_path / f"{i}.co"
        obj.write_bytes(code)
        text = subprocess.run([OBJDUMP, "-d", "--mcpu=gfx950", str(obj)], check=True, capture_output=True, text=True).stdout
        f, n = hazards(text.splitlines())
        found += f
        loads += n
    assert loads > 100
    assert not found, f"{len(found)} of {loads} loads, the first: {found[0]}"
