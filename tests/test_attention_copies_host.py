"""The attention kernels copy their tiles to LDS by instructions that the compiler's hazard tables know nothing of.  In the code built for the GPU every
such copy brings the wait states itself that a buffer load needs behind a vector instruction that wrote one of its scalar registers (five)."""
import os
import re
import subprocess

from paper_2405_01248_amd import build

WAIT_STATES = 5


def test_every_copy_to_lds_brings_its_wait_states(tmp_path):
    out = str(tmp_path / "attention.s")
    flags = [f for f in build.FLAGS if f not in ("-fPIC", "-Wall", "-Wno-unused-function")]
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), *flags, "--cuda-device-only", "-S", os.path.join(build.CSRC, "attention.hip"), "-o", out],
                   check=True, stdout=subprocess.DEVNULL, stderr=subprocess.DEVNULL)
    copies, bad, inside, states, m0 = 0, [], False, 0, False
    for n, line in enumerate(open(out).read().splitlines()):
        if "#ASMSTART" in line:
            inside, states, m0 = True, 0, False
        code = line.split(";")[0].strip()
        if "#ASMEND" in line:
            inside = False
        elif re.match(r"buffer_load_\S+ .*\blds$", code):
            copies += 1
            if not (inside and m0 and states >= WAIT_STATES):
                bad.append((n, line, states))
        elif code and not code.startswith("."):
            states += 1 + (int(code.split()[1]) if code.startswith("s_nop") else 0)
            # (a vector instruction in front of the copy, behind the wait states, would need them again)
            if code.startswith("v_"):
                states = 0
            m0 = m0 or code.startswith("s_mov_b32 m0,")
    assert copies > 0 and not bad, (copies, bad[:10])
