"""Wait states around the inline assembly of the bf16 kernels, in the listing that the build's compiler writes.  The
compiler inserts the wait states of gfx9 between its own instructions but not before those of inline assembly:

* five between a vector instruction that writes a scalar register and a memory instruction that reads it;
* one between a write of M0 and an LDS DMA;
* up to nineteen between an MFMA and a vector instruction that reads its result, so inline assembly holds no
  vector instruction (empty statements that only pin a register are no instructions)."""

import os
import re
import subprocess

import pytest

from paper_2606_10537_amd import build as B

SRC = "attn_bf16.hip"
MEM = ("global_", "buffer_", "flat_", "scratch_")


def regs(text):
    out = [int(x) for x in re.findall(r"(?<![\w\[])s(\d+)\b", text)]
    for a, b in re.findall(r"\bs\[(\d+):(\d+)\]", text):
        out += range(int(a), int(b) + 1)
    return out


def check(lines):
    """Violations in a listing, textual order; a scalar instruction that rewrites a register clears it."""
    bad, dmas, t, written, m0, in_asm = [], 0, 0, {}, -99, False
    for line in lines:
        s = line.strip()
        if "#ASMSTART" in s or "#ASMEND" in s:
            in_asm = "#ASMSTART" in s
            continue
        if re.match(r"^_Z\w+:", s):
            written, m0 = {}, -99
        if not re.match(r"^(s_|v_|ds_|global_|buffer_|flat_|scratch_)\w", s):
            continue
        op, _, args = s.partition(" ")
        dst, _, src = args.partition(",")
        if in_asm and op.startswith("v_"):
            bad.append(f"vector instruction in inline assembly: {s}")
        if op.startswith(MEM):
            for r in regs(args):
                if t - written.get(r, -99) - 1 < 5:
                    bad.append(f"{s}: s{r} written by a vector instruction {t - written[r] - 1} wait states before")
            if op.startswith("global_load_lds"):
                dmas += 1
                if t - m0 - 1 < 1:
                    bad.append(f"{s}: M0 written just before")
        if op.startswith("v_"):
            for r in regs(dst):
                written[r] = t
        elif op.startswith("s_"):
            for r in regs(dst):
                written.pop(r, None)
            if dst.strip() == "m0":
                m0 = t
        t += int(args) + 1 if op == "s_nop" else 1
    return bad, dmas


def test_each_rule():
    lds = "global_load_lds_dwordx4 v1, s[4:5]"
    assert check(["v_readfirstlane_b32 s5, v2", "s_mov_b32 m0, s9", "s_nop 3", lds]) == ([], 1)
    assert len(check(["v_readfirstlane_b32 s5, v2", "s_mov_b32 m0, s9", "s_nop 2", lds])[0]) == 1
    assert len(check(["s_mov_b32 m0, s9", lds])[0]) == 1
    assert check(["v_readfirstlane_b32 s5, v2", "s_mov_b64 s[4:5], s[6:7]", "s_nop 0", lds]) == ([], 1)
    asm = [";;#ASMSTART", "v_max_f32 v1, v2, v3", ";;#ASMEND"]
    assert len(check(asm)[0]) == 1


@pytest.mark.parametrize("defines", [[], ["-DPD_CHECK_INDICES=1"]], ids=["release", "checking"])
def test_listing(tmp_path, defines):
    if not os.path.exists(B.HIPCC):
        pytest.skip(f"no compiler at {B.HIPCC}")
    out = tmp_path / "attn.s"
    r = subprocess.run([B.HIPCC, *B.FLAGS, *B.EXTRA.get(SRC, []), *defines, "--cuda-device-only", "-S",
                        os.path.join(B.CSRC, SRC), "-o", str(out)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]
    bad, dmas = check(out.read_text().splitlines())
    assert dmas > 100
    assert not bad, f"{len(bad)}: " + "; ".join(bad[:5])
