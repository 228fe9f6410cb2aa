"""The weight-gradient tiles read LDS through inline assembly that the compiler's own waits know nothing of.  In the code built for the GPU no
branch is taken, and no register of theirs is read, with such a load outstanding: what happens on the other side of a branch (a register
copied on the way into a loop, say) may need the value."""
import os
import re
import subprocess

from paper_2405_01248_amd import build


def _listing(tmp_path):
    out = str(tmp_path / "gemm_dw.s")
    flags = [f for f in build.FLAGS if f not in ("-fPIC", "-Wall", "-Wno-unused-function")]
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), *flags, "--cuda-device-only", "-S", os.path.join(build.CSRC, "gemm_dw.hip"), "-o", out],
                   check=True, stdout=subprocess.DEVNULL, stderr=subprocess.DEVNULL)
    return open(out).read().splitlines()


def _registers(text):
    regs = set()
    for lo, hi, one in re.findall(r"\bv\[(\d+):(\d+)\]|\bv(\d+)\b", text):
        regs.update(range(int(lo), int(hi) + 1) if lo else [int(one)])
    return regs


def test_no_branch_and_no_use_with_a_transposing_load_outstanding(tmp_path):
    outstanding, loads, bad = set(), 0, []
    for n, line in enumerate(_listing(tmp_path)):
        code = line.split(";")[0].strip()
        if not code or code.startswith("."):
            if outstanding and re.match(r"\.LBB\d+_\d+:", code):
                bad.append((n, line))
            continue
        op, _, args = code.partition(" ")
        if op == "ds_read_b64_tr_b16":
            loads += 1
            outstanding |= _registers(args.split(",")[0])
        elif op == "s_waitcnt" and "lgkmcnt(0)" in args:
            outstanding = set()
        elif outstanding and (op.startswith(("s_cbranch", "s_branch")) or (op.startswith("v_") and _registers(args) & outstanding)):
            bad.append((n, line))
    assert loads > 0 and not bad, bad[:10]
