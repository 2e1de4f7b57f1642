"""Wait states that the compiler cannot put inside an inline-assembly block, checked in the built gfx950 code of both libraries: a
direct-to-LDS load takes its LDS address from M0 and must not directly follow the scalar instruction that writes M0 (one wait
state; without it the load may land at the previous load's address)."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2602_05305_amd import build as fb_build

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


def _instructions(lib, tmp_path):
    """[(function, instruction text)] of every gfx950 code object in the library, in program order."""
    shutil.copy(lib, tmp_path)
    name = os.path.basename(lib)
    subprocess.run([OBJDUMP, "--offloading", name], cwd=tmp_path, check=True, capture_output=True)
    out = []
    for f in sorted(os.listdir(tmp_path)):
        if not (f.startswith(name + ".") and f.endswith("gfx950")):
            continue
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", f], cwd=tmp_path, check=True, capture_output=True, text=True).stdout
        func = ""
        for line in text.splitlines():
            label = re.match(r"^[0-9a-f]+ <(.+)>:", line)
            if label:
                func = label.group(1)
            elif line.startswith("\t"):
                out.append((func, line.split("//")[0].strip()))
    return out


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no disassembler in this installation")
@pytest.mark.parametrize("lib", [fb_build.LIB, fb_build.CALIB_LIB])
def test_direct_to_lds_load_waits_for_m0(lib, tmp_path):
    if not os.path.exists(lib):
        fb_build.build(force=True)
    ins = _instructions(lib, tmp_path)
    loads, early = 0, []
    for (_, before), (func, text) in zip(ins, ins[1:]):
        if re.match(r"(global|scratch|buffer)_load_lds_|buffer_load_\w+ .*\blds\b", text):
            loads += 1
            if re.match(r"s_\w+ m0\b", before):
                early.append(f"{func}: {before}; {text}")
    assert loads > 0
    assert not early, f"{len(early)} of {loads} loads, first: {early[0]}"
