"""CPU test of the compiled device code: wait states that gfx950 leaves to the
program."""
import os
import re
import struct
import subprocess

import pytest

from paper_2606_24033_amd import blockgtq as bg
from paper_2606_24033_amd import build as b

OBJDUMP = os.path.join(os.path.dirname(os.path.realpath(b.HIPCC)), "..", "llvm", "bin", "llvm-objdump")
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"
TRANS = re.compile(r"v_(exp|log|rcp|rcp_iflag|rsq|sqrt|sin|cos)_(f16|f32|f64|bf16)")


def code_objects(path):
    """The gfx950 code objects of the library: one uncompressed offload bundle
    per source file, each a table of (offset, size, target) entries."""
    data = open(path, "rb").read()
    for m in re.finditer(re.escape(MAGIC), data):
        at = m.start() + len(MAGIC)
        (n,) = struct.unpack_from("<Q", data, at)
        if not 0 < n < 16:  # the name in a string table, not a bundle
            continue
        at += 8
        for _ in range(n):
            off, size, length = struct.unpack_from("<QQQ", data, at)
            target = data[at + 24:at + 24 + length]
            at += 24 + length
            if b"gfx950" in target and size:
                yield data[m.start() + off:m.start() + off + size]


def vgprs(operand):
    m = re.search(r"\bv\[(\d+):(\d+)\]", operand)
    if m:
        return set(range(int(m.group(1)), int(m.group(2)) + 1))
    m = re.search(r"\bv(\d+)\b", operand)
    return {int(m.group(1))} if m else set()


def unguarded(lines):
    """Plain VALU instructions directly behind a transcendental one whose
    result they read."""
    kernel, result = "", None
    for line in lines:
        head = re.match(r"[0-9a-f]+ <(\S+)>:", line)
        if head:
            kernel, result = head.group(1), None
        text = line.split("//")[0].strip()
        if head or not text:
            continue
        name, _, rest = text.partition(" ")
        ops = rest.split(",")
        if result and name.startswith("v_") and not TRANS.match(name):
            # (compares name no vector destination, the mixhi form keeps half of its own)
            reads = ops if name.startswith(("v_cmp", "v_fma_mixhi")) else ops[1:]
            if any(result & vgprs(o) for o in reads):
                yield f"{kernel}: {text}"
        result = vgprs(ops[0]) if TRANS.match(name) else None


def test_wait_state_after_transcendental_instructions(tmp_path):
    """gfx950 needs one wait state between a transcendental instruction and a
    plain VALU instruction that reads its result.  The compiler keeps it for
    its own instructions but does not look into inline asm."""
    if not os.path.exists(OBJDUMP):
        pytest.skip("no llvm-objdump beside hipcc")
    objects = list(code_objects(bg.LIB_PATH))
    assert len(objects) == sum(s.endswith(".hip") for s in b.SOURCES)
    seen, bad = 0, []
    for i, obj in enumerate(objects):
        path = tmp_path / f"{i}.co"
        path.write_bytes(obj)
        lines = subprocess.run([OBJDUMP, "-d", str(path)], capture_output=True, text=True, check=True).stdout.splitlines()
        seen += sum("v_exp_f32" in x for x in lines)
        bad += unguarded(lines)
    assert seen > 0
    assert not bad, "\n".join(bad[:20])
