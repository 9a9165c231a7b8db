"""Inline assembly of the prefill kernels: the compiler neither sees what it reads and writes late nor inserts wait states around
it.  The assembly that the build's compiler makes of these kernels is scanned for what must not stand next to a statement:
  - a vector instruction that writes an operand of an MFMA less than 2 wait states before it;
  - a reader or writer of an MFMA's result less than 12 wait states behind it, other MFMAs apart;
  - a vector instruction that writes a scalar of a copy's descriptor less than 5 wait states before the copy, or M0 less than 1;
  - an MFMA that writes what a store of 16 bytes reads less than 18 wait states before it, or an instruction that writes its data less than 2 behind it.
Every instruction counts as one wait state (s_nop N as N + 1, an MFMA of four passes as four); along the text, not along branches."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2602_06072_amd import build


def registers(kind, text):
    out = set()
    for a, b, c in re.findall(rf"(?<![a-z0-9_]){kind}(?:\[(\d+):(\d+)\]|(\d+))", text):
        out |= {int(c)} if c else set(range(int(a), int(b) + 1))
    return out


def instructions(text):
    """[(op, operands, in inline assembly)]"""
    out, own = [], False
    for line in text.splitlines():
        if "#ASMSTART" in line or "#ASMEND" in line:
            own = "#ASMSTART" in line
        m = re.match(r"\s+([a-z]\w+)\s*([^;]*)", line)
        if m and not line.strip().startswith("."):
            out.append((m[1], [x.strip() for x in m[2].split(",")], own))
    return out


def wait_states(op, args):
    return int(args[0], 0) + 1 if op == "s_nop" else 4 if op.startswith("v_mfma") else 1


def hazards(text):
    code, found, stores = instructions(text), [], 0
    for i, (op, args, own) in enumerate(code):
        mfma, copy = own and op.startswith("v_mfma"), own and op.startswith("buffer_load") and args[-1].endswith("lds")
        if own and op == "global_store_dwordx4":
            stores += 1
            reads, data = registers("v", " ".join(args[:2])), registers("v", args[1])
            gone, j = 0, i - 1
            while j >= 0 and gone < 18:
                o, a, _ = code[j]
                if o.startswith("v_mfma") and registers("v", a[0]) & reads:
                    found.append(("written by an MFMA before", o, a, op, args))
                gone, j = gone + wait_states(o, a), j - 1
            gone, j = 0, i + 1
            while j < len(code) and gone < 2 and code[j][0] not in ("s_branch", "s_endpgm", "s_setpc_b64"):
                o, a, _ = code[j]
                if o.startswith(("v_", "ds_read", "buffer_load", "global_load")) and registers("v", " ".join(a[:2] if "swap" in o else a[:1])) & data:
                    found.append(("data written behind", o, a, op, args))
                gone, j = gone + wait_states(o, a), j + 1
        if not (mfma or copy):
            continue
        reads = registers("v", " ".join(args[1:4])) if mfma else registers("s", " ".join(args[1:2]))
        gone, j = 0, i - 1
        while j >= 0 and gone < (2 if mfma else 5):
            o, a, _ = code[j]
            if o.startswith("v_") and not o.startswith("v_mfma"):
                written = registers("v" if mfma else "s", " ".join(a[:2] if "swap" in o else a[:1]))
                if written & reads:
                    found.append(("written right before", o, a, op, args))
            if copy and gone < 1 and o.startswith("s_") and a[0] == "m0":
                found.append(("M0 right before", o, a, op, args))
            gone, j = gone + wait_states(o, a), j - 1
        gone, j = 0, i + 1
        while mfma and j < len(code) and gone < 12:
            o, a, _ = code[j]
            if o in ("s_branch", "s_endpgm", "s_setpc_b64"):
                break
            if not o.startswith("v_mfma") and registers("v", " ".join(a)) & registers("v", args[0]):
                found.append(("used right behind", o, a, op, args))
            gone, j = gone + wait_states(o, a), j + 1
    return found, sum(own and op.startswith("v_mfma") for op, _, own in code), sum(own and op.startswith("buffer_load") for op, _, own in code), stores


MFMA = "\t;;#ASMSTART\n\tv_mfma_f32_16x16x32_bf16 v[8:11], v[0:3], v[4:7], v[8:11]\n\t;;#ASMEND\n"
STORE = "\t;;#ASMSTART\n\tglobal_store_dwordx4 v[2:3], v[4:7], off sc1{}\n\t;;#ASMEND\n"
COPY = "\t;;#ASMSTART\n\tbuffer_load_dwordx4 v1, s[4:7], 0 offen lds\n\t;;#ASMEND\n"


@pytest.mark.parametrize("before, statement, behind, n", [
    ("\tv_mov_b32_e32 v5, v20\n", MFMA, "", 1), ("\tv_mov_b32_e32 v5, v20\n\ts_nop 1\n", MFMA, "", 0), ("\tv_mov_b32_e32 v12, v5\n", MFMA, "", 0),
    ("", MFMA, "\ts_nop 10\n\tv_add_f32_e32 v20, v9, v20\n", 1), ("", MFMA, "\ts_nop 11\n\tv_add_f32_e32 v20, v9, v20\n", 0),
    ("", MFMA, MFMA * 3 + "\tds_write_b64 v30, v[10:11]\n", 3), ("\tv_readlane_b32 s5, v9, 3\n\ts_nop 3\n", COPY, "", 1),
    ("\tv_readlane_b32 s5, v9, 3\n\ts_nop 4\n", COPY, "", 0), ("\ts_mov_b32 m0, s9\n", COPY, "", 1), ("\ts_mov_b32 m0, s9\n\ts_nop 0\n", COPY, "", 0),
    ("", STORE.format("\n\ts_nop 1"), "\tv_mov_b32_e32 v5, v20\n", 0), ("", STORE.format("\n\ts_nop 0"), "\tv_mov_b32_e32 v5, v20\n", 1), ("", STORE.format(""), "\tds_read_b128 v[6:9], v1\n", 1),
    ("", STORE.format(""), "\tv_mov_b32_e32 v2, v20\n", 0), ("\tv_mfma_f32_16x16x32_bf16 v[4:7], v[20:23], v[24:27], v[4:7]\n\ts_nop 12\n", STORE.format("\n\ts_nop 1"), "", 1),
    ("\tv_mfma_f32_16x16x32_bf16 v[4:7], v[20:23], v[24:27], v[4:7]\n\ts_nop 15\n\ts_nop 1\n", STORE.format("\n\ts_nop 1"), "", 0)])
def test_the_scan_finds_what_is_planted(before, statement, behind, n):
    assert len(hazards(before + statement + behind)[0]) == n      # (of the four MFMAs the first is twelve wait states away)


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")
@pytest.mark.parametrize("src", sorted(build.NO_SCALAR_SPILLS))
def test_no_hazard_next_to_inline_assembly(src, tmp_path):
    out = str(tmp_path / "kernel.s")
    subprocess.run(["hipcc", *build.HIP_FLAGS, "-S", "--cuda-device-only", os.path.join(build.CSRC, src), "-o", out], check=True, capture_output=True)
    found, mfmas, copies, stores = hazards(open(out).read())
    assert mfmas > 300 and copies > 100 and stores > 30     # (the pipelined kernels of both head dimensions; the others' outputs)
    assert not found, found[:5]
