"""No store of more than eight bytes has its data overwritten by the instruction after it (no GPU:
the sources are searched, and a kernel is compiled to assembly here).

A 16-byte buffer store with part of its offset in a scalar register was followed directly by a
vector instruction that wrote the first of its data registers: now and then four lanes of every
sixteen stored the new value (steps with separate reverse inputs, 129 to 256 tokens, dstate 16 and
32, more than 256 row-heads: columns 32, 36, 40 and 44 of tokens 236 to 239).  After stores with a
constant offset the compiler leaves a wait state; after those it does not.
"""
import glob
import os
import re

import pytest

from paper_2607_02805_amd import build
from tests.test_mfma_chains import _compile_to_asm

SOURCES = sorted(glob.glob(os.path.join(build.CSRC, "*.hip")))


def regs(tok):
    """(register file, index) of every register of an operand."""
    m = re.match(r"([va])\[(\d+):(\d+)\]$", tok) or re.match(r"([va])(\d+)$", tok)
    return {(m[1], i) for i in range(int(m[2]), int(m[m.lastindex]) + 1)} if m else set()


def overwritten_stores(asm):
    """(function, store, next instruction) where the next instruction writes the store's data."""
    found, fn, last = [], None, None
    for line in asm.splitlines():
        line = line.split(";")[0].strip()
        m = re.match(r"(_Z\w+):", line)
        if m or line.endswith(":"):
            fn, last = (m[1] if m else fn), (None if m else last)
        if not line or line.startswith(".") or line.endswith(":"):
            continue
        op, _, rest = line.partition(" ")
        ops = [o.strip() for o in rest.split(",")]
        if last and op.startswith("v_") and regs(ops[0]) & last[1]:
            found.append((fn, last[0], line))
        last = None
        if re.match(r"(buffer|global|flat|scratch)_store_dwordx[34]$", op):
            last = (line, regs(ops[0 if op.startswith("buffer") else 1]))
    return found


def calls(text, name):
    """The argument lists of every call of ``name``."""
    for m in re.finditer(name + r"\(", text):
        depth, args, cur = 1, [], ""
        for ch in text[m.end():]:
            depth += (ch in "([{") - (ch in ")]}")
            if depth == 0:
                break
            if ch == "," and depth == 1:
                args.append(cur.strip())
                cur = ""
            else:
                cur += ch
        yield args + [cur.strip()]


@pytest.mark.parametrize("src", SOURCES, ids=os.path.basename)
def test_wide_buffer_stores_have_no_scalar_offset(src):
    for args in calls(open(src).read(), r"raw_buffer_store_b(?:96|128)"):
        assert args[3] == "0", args


def test_compiled_stores_keep_their_data(tmp_path):
    if not os.path.exists(build.HIPCC):
        pytest.skip("hipcc not available")
    out = str(tmp_path / "k.s")
    _compile_to_asm("bdlm_maskw.hip", out)
    asm = open(out).read()
    assert "buffer_store_dwordx4" in asm
    assert overwritten_stores(asm) == []


def test_the_scan_finds_a_planted_overwrite():
    head = "_ZN4bdlm1fEv:\n"
    bad = head + "\tbuffer_store_dwordx4 v[22:25], v66, s[4:7], s0 offen\n\tv_and_b32_e32 v22, 0xffff0000, v45\n"
    assert len(overwritten_stores(bad)) == 1
    assert overwritten_stores(bad.replace("\tv_and", "\ts_nop 0\n\tv_and")) == []
    assert overwritten_stores(bad.replace("v22, 0xffff", "v26, 0xffff")) == []
    assert overwritten_stores(bad.replace("v[22:25]", "a[22:25]")) == []
    glob_ = head + "\tglobal_store_dwordx4 v[2:3], v[4:7], off\n\tv_mov_b32_e32 v7, 0\n"
    assert len(overwritten_stores(glob_)) == 1
    assert overwritten_stores(glob_.replace("v7, 0", "v2, 0")) == []
