"""Properties of the built gfx950 code that the sources ask for and the compiler can lose.

A direct-to-LDS load takes its LDS address from M0 and must not directly follow the scalar instruction that writes M0 (one wait state,
which the compiler cannot put inside an inline-assembly block; without it the load may land at the previous load's address).

The dense streaming passes store split partials non-temporally and the final partial of an unsplit pass normally; where the two
stores share code, they are merged and the hint is gone."""
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


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no disassembler in this installation")
def test_split_partials_are_stored_non_temporally(tmp_path):
    if not os.path.exists(fb_build.LIB):
        fb_build.build(force=True)
    stores = {}
    for func, text in _instructions(fb_build.LIB, tmp_path):
        kernel = re.search(r"attn_stream_kernelILi(64|128)ELi([04])ELi\dELi\dE", func)      # modes: dense, per-head refresh
        if kernel and text.startswith("global_store_dwordx4"):
            n = stores.setdefault(func, [0, 0])
            n[text.endswith(" nt")] += 1
    assert len(stores) >= 20
    for func, (plain, hinted) in stores.items():
        assert plain == hinted, f"{func}: {hinted} of {plain + hinted} row stores are non-temporal"


def _vector_registers(operand):
    m = re.fullmatch(r"(-?\|?)([va])(?:(\d+)|\[(\d+):(\d+)\])\|?", operand.strip())
    if not m:
        return set()
    first = int(m.group(3) if m.group(3) else m.group(4))
    return {(m.group(2), r) for r in range(first, (first if m.group(3) else int(m.group(5))) + 1)}


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no disassembler in this installation")
@pytest.mark.parametrize("lib", [fb_build.LIB, fb_build.CALIB_LIB])
def test_products_read_what_vector_instructions_wrote_two_wait_states_later(lib, tmp_path):
    """The hardware does not wait by itself; the compiler keeps the distance for the instructions it knows, not for the results of
    inline assembly."""
    if not os.path.exists(lib):
        fb_build.build(force=True)
    ins = _instructions(lib, tmp_path)
    products, early = 0, []
    for i, (func, text) in enumerate(ins):
        if not text.startswith("v_mfma"):
            continue
        products += 1
        operands = text.split(None, 1)[1].split(",")
        reads = set().union(*(_vector_registers(x) for x in operands[1:4]))
        waited = 0
        for back, before in reversed(ins[max(0, i - 2):i]):
            if back != func or waited >= 2:
                break
            nop = re.match(r"s_nop (\d+)", before)
            if before.startswith("v_") and not before.startswith("v_mfma") and " " in before:
                written = before.split(None, 1)[1].split(",")[:2 if "swap" in before else 1]
                if reads & set().union(*(_vector_registers(x) for x in written)):
                    early.append(f"{func}: {before}, {waited} wait states, {text}")
            waited += int(nop.group(1)) + 1 if nop else 1
    assert products > 0
    assert not early, f"{len(early)} places, first: {early[0]}"
