"""No vector instruction of the built kernels stands between the join of an `if`
and the instruction that gives its lanes back (no GPU: the library is
disassembled).

The compiler has placed stores of spilled registers there: `s_and_saveexec s[a:b]`
/ `s_cbranch_execz L` ... `L:` spill stores, then `s_or exec, exec, s[a:b]`.  The
stores run for the lanes of the `if` alone, and what the other lanes held (sums,
halves of addresses) is lost.  It happened in kernels with hardly a register to
spare, in some shapes only, and no source shows it."""
import os
import re
import struct
import subprocess

import pytest

LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2609_31093_amd", "libpisa.so")
OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def code_objects(blob):
    """The gfx950 code objects of every offload bundle in the library."""
    at = blob.find(MAGIC)
    while at >= 0:
        n, = struct.unpack_from("<Q", blob, at + len(MAGIC))
        o = at + len(MAGIC) + 8
        for _ in range(n):
            off, size, length = struct.unpack_from("<QQQ", blob, o)
            ident = blob[o + 24:o + 24 + length].decode()
            o += 24 + length
            if "gfx950" in ident and size:
                yield blob[at + off:at + off + size]
        at = blob.find(MAGIC, at + 1)


def early_instructions(asm):
    """(kernel, label, instructions) of every join whose lanes come back late."""
    found, kernels = [], 0
    for part in re.split(r"\n(?=<_Z)", asm)[1:]:
        kernels += 1
        name = part[1:part.index(">")]
        lines = [l.split("//")[0].strip() for l in part.splitlines()[1:]]
        label = {l[1:-2]: i for i, l in enumerate(lines) if re.fullmatch(r"<L\d+>:", l)}
        for i, line in enumerate(lines):
            m = re.fullmatch(r"s_cbranch_execz (L\d+)", line)
            if not m or m.group(1) not in label:
                continue
            saved = None
            for j in range(i - 1, max(-1, i - 12), -1):
                s = re.match(r"s_and_saveexec_b64 (s\[\d+:\d+\]|vcc)", lines[j])
                if s or lines[j].endswith(">:"):
                    saved = s and s.group(1)
                    break
            if not saved:
                continue
            early = []
            for x in lines[label[m.group(1)] + 1:]:
                if x == f"s_or_b64 exec, exec, {saved}":
                    if early:
                        found.append((name, m.group(1), early))
                    break
                if x.endswith(">:") or re.match(r"s_c?branch|s_endpgm", x):
                    break
                if re.match(r"v_|scratch_|global_|buffer_|flat_|ds_", x) and not re.match(
                        r"v_readlane|v_writelane|v_readfirstlane", x):
                    early.append(x)
    return kernels, found


def test_scan_finds_a_store_before_the_restore():
    text = """
<_Zk>:
	s_and_saveexec_b64 s[2:3], vcc
	s_cbranch_execz L0
	v_mov_b32_e32 v1, v2
<L0>:
	s_waitcnt vmcnt(0)
	scratch_store_dword off, v5, off offset:4
	s_or_b64 exec, exec, s[2:3]
	s_endpgm
"""
    assert early_instructions(text) == (1, [("_Zk", "L0", ["scratch_store_dword off, v5, off offset:4"])])
    fine = text.replace("\tscratch_store_dword off, v5, off offset:4\n", "")
    assert early_instructions(fine) == (1, [])


def test_lanes_come_back_before_anything_else(tmp_path):
    if not (os.path.exists(LIB) and os.path.exists(OBJDUMP)):
        pytest.skip("needs the built library and llvm-objdump")
    with open(LIB, "rb") as f:
        blob = f.read()
    total, found = 0, []
    for i, code in enumerate(code_objects(blob)):
        path = tmp_path / f"{i}.co"
        path.write_bytes(code)
        asm = subprocess.run([OBJDUMP, "-d", "--symbolize-operands", "--no-show-raw-insn", "--no-leading-addr", str(path)],
                             check=True, capture_output=True, text=True).stdout
        kernels, early = early_instructions(asm)
        total += kernels
        found += early
    assert total > 100  # the library's kernels were seen
    assert not found, found
