"""The GPU code inside the built library: what its kernels take, and their listing."""
import os
import re
import struct
import subprocess

from paper_2405_01248_amd import build

LLVM = "/opt/rocm/llvm/bin"
_MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def code_objects(tmp_path):
    """The gfx950 code object of each source with kernels, as files."""
    fat = str(tmp_path / "fat.bin")
    subprocess.run([os.path.join(LLVM, "llvm-objcopy"), f"--dump-section=.hip_fatbin={fat}", build.LIB, os.devnull], check=True)
    with open(fat, "rb") as f:
        data = f.read()
    out, at = [], data.find(_MAGIC)
    while at >= 0:
        count, pos = struct.unpack_from("<Q", data, at + 24)[0], at + 32
        for _ in range(count):
            offset, size, name_len = struct.unpack_from("<QQQ", data, pos)
            name = data[pos + 24:pos + 24 + name_len]
            pos += 24 + name_len
            if b"gfx950" in name and size:
                out.append(str(tmp_path / f"{len(out)}.co"))
                with open(out[-1], "wb") as f:
                    f.write(data[at + offset:at + offset + size])
        at = data.find(_MAGIC, at + 24)
    return out


def resources(code_object):
    """{mangled kernel name: {"private_segment_fixed_size": .., "vgpr_count": .., "vgpr_spill_count": .., "sgpr_spill_count": ..}}"""
    notes = subprocess.run([os.path.join(LLVM, "llvm-readelf"), "--notes", code_object], check=True, capture_output=True, text=True).stdout
    out = {}
    for kernel in re.split(r"\n\s+- \.agpr_count", notes)[1:]:
        field = lambda name: re.search(rf"\.{name}:\s*(\S+)", kernel).group(1)  # noqa: E731
        out[field("symbol").strip("'").removesuffix(".kd")] = {n: int(field(n)) for n in ("private_segment_fixed_size", "vgpr_count", "vgpr_spill_count", "sgpr_spill_count")}
    return out


def listings(code_object, wanted):
    """(mangled kernel name, its instructions) of the kernels whose name `wanted` accepts."""
    names = [n for n in resources(code_object) if wanted(n)]
    if not names:
        return
    text = subprocess.run([os.path.join(LLVM, "llvm-objdump"), "-d", "--no-show-raw-insn", "--disassemble-symbols=" + ",".join(names), code_object],
                          check=True, capture_output=True, text=True).stdout
    for part in re.split(r"\n[0-9a-f]+ <", text)[1:]:
        name, _, body = part.partition(">:")
        yield name, [line.split("//")[0].strip() for line in body.splitlines() if line.strip()]
