"""Wait states in the machine code of the kernels (no GPU: the sources are
compiled to assembly here and the listing is read).

Between a vector instruction that writes a scalar register and a vector
instruction that reads it, and between a matrix product and the first read of
its result, the hardware needs wait states that the compiler inserts -- but not
in front of inline asm.  So no asm instruction may come closer than two wait
states to the vector instruction that wrote its scalar operand, and none may be
the first to read a product's result.
"""
import functools
import os
import re
import subprocess

import pytest

from paper_2305_00515_amd import build


def registers(text, kind):
    """Numbers of the registers of `kind` (v or s) that an operand list names."""
    out = set()
    for m in re.finditer(r"(?<![\w])%s(?:(\d+)|\[(\d+):(\d+)\])" % kind, text):
        out |= set(range(int(m[1]), int(m[1]) + 1) if m[1] else range(int(m[2]), int(m[3]) + 1))
    return out


def findings(listing):
    bad = []
    where, asm = "?", False
    written = {}       # scalar register -> wait states since a vector instruction wrote it
    products = []      # result registers of products that no compiled instruction has read yet
    for line in listing.splitlines():
        s = line.strip()
        if s.startswith(";"):
            asm = "#ASMSTART" in s or (asm and "#ASMEND" not in s)
            continue
        m = re.match(r"(\S+):\s*;\s*@", line)
        if m:
            where, written, products = m[1], {}, []
            continue
        s = s.split(";")[0].strip()
        if not s or s[0] == "." or s.endswith(":"):
            continue
        op, _, rest = s.partition(" ")
        dst, _, src = rest.partition(",")
        if op.startswith("v_"):
            late = registers(src, "s") & set(written)
            if (asm or op == "v_writelane_b32") and late:
                bad.append("%s: %s after %d wait state(s)" % (where, s, min(written[r] for r in late)))
            read = registers(rest if op in ("v_writelane_b32",) else src, "v")
            if op.startswith("v_mfma"):
                products.append(registers(dst, "v"))
            else:
                hit = [p for p in products if p & read]
                if asm and hit:
                    bad.append("%s: %s reads a product first" % (where, s))
                products = [p for p in products if p not in hit]
        states = int(rest) + 1 if op == "s_nop" else 1
        written = {r: n + states for r, n in written.items() if n + states < 2}
        if op.startswith("v_"):
            written.update((r, 0) for r in registers(dst, "s"))
    return bad


def test_reader_finds_what_it_looks_for():
    head = "k: ; @k\n"
    asm = "\t;;#ASMSTART\n\tv_mad_i32_i24 v1, v2, s3, v4\n\t;;#ASMEND\n"
    assert findings(head + "v_readlane_b32 s3, v9, 7\n" + asm)
    assert findings(head + "v_readlane_b32 s3, v9, 7\ns_nop 0\n" + asm)
    assert not findings(head + "v_readlane_b32 s3, v9, 7\ns_nop 1\n" + asm)
    assert findings(head + "v_readlane_b32 s3, v9, 7\nv_mov_b32 v8, 0\nv_writelane_b32 v1, s3, 19\n")
    assert findings(head + "v_mfma_i32_16x16x64_i8 v[2:5], v[10:13], v[14:17], 0\n" + asm)
    assert not findings(head + "v_mfma_i32_16x16x64_i8 v[2:5], v[10:13], v[14:17], 0\nv_mul_i32_i24 v6, v3, v3\n" + asm)


@functools.lru_cache(None)
def listing_of(source):
    """The assembly of a kernel source."""
    try:
        build.hipcc()
    except RuntimeError:
        pytest.skip("no hipcc")
    flags = [f for f in build.FLAGS if f not in ("-shared", "-fPIC")]
    return subprocess.run([build.hipcc()] + flags + ["-S", "--cuda-device-only", "-o", "-",
                                                     os.path.join(build.CSRC, source)],
                          check=True, capture_output=True, text=True).stdout


@pytest.mark.parametrize("source", [s for s in build.SOURCES if s.endswith(".hip")])
def test_no_asm_before_its_operand_is_ready(source):
    bad = findings(listing_of(source))
    assert not bad, "%d places, e.g. %s" % (len(bad), bad[:3])
