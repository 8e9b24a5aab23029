"""What the built device code has to keep to.

Wait states: a vector memory instruction that
reads a scalar register needs five wait states after a vector instruction
wrote it (v_readlane, v_readfirstlane, a compare): the compiler pads its own
loads, but does not see the buffer copies written in assembly, whose operands
it may have reloaded from a spill lane just before.

Registers: the softmax with eight waves a workgroup is chosen so that two
workgroups share a CU, which 16 waves of at most 128 registers do."""
import os
import re
import shutil
import subprocess

import pytest

PATH = "/opt/rocm/llvm/bin:" + os.environ.get("PATH", "")
OBJDUMP = shutil.which("llvm-objdump", path=PATH)
READELF = shutil.which("llvm-readelf", path=PATH)
WAITS = 5


def _scalars(text):
    """Numbers of the scalar registers named in an operand text."""
    out = set()
    for lo, hi in re.findall(r"\bs\[(\d+):(\d+)\]", text):
        out.update(range(int(lo), int(hi) + 1))
    out.update(int(n) for n in re.findall(r"\bs(\d+)\b", text))
    return out


def short_waits(lines):
    """(kernel, line) of each buffer access too close to the vector
    instruction that wrote one of its scalar registers."""
    bad, kernel, recent = [], "", []  # recent: (wait states it counts for, scalars it wrote)
    for line in lines:
        m = re.match(r"^[0-9a-f]+ <(.*)>:$", line)
        if m:
            kernel, recent = m.group(1), []
            continue
        ins = line.split("//")[0].strip()
        if not ins:
            continue
        op, _, args = ins.partition(" ")
        if op.startswith("buffer_"):
            used, waited = _scalars(args), 0
            for states, wrote in reversed(recent):
                if waited >= WAITS:
                    break
                if used & wrote:
                    bad.append((kernel, ins))
                    break
                waited += states
        states = int(args, 0) + 1 if op == "s_nop" else 1
        wrote = _scalars(args.split(",")[0]) if op.startswith("v_") else set()
        if op.startswith(("v_add_co", "v_sub_co", "v_addc_co", "v_div_scale")):
            wrote |= _scalars(",".join(args.split(",")[:2]))
        recent = (recent + [(states, wrote)])[-WAITS:]
    return bad


def test_scan_counts_wait_states():
    head = ["0000000000000000 <k>:", "\tv_readlane_b32 s7, v1, 3"]
    load = ["\tbuffer_load_dwordx4 v2, s[4:7], s2 offen lds"]
    assert len(short_waits(head + ["\ts_mov_b32 m0, s3", "\ts_nop 0"] + load)) == 1
    assert not short_waits(head + ["\ts_mov_b32 m0, s3", "\ts_nop 3"] + load)
    assert not short_waits(["0000000000000000 <k>:", "\tv_readlane_b32 s8, v1, 3"] + load)
    assert len(short_waits(head + ["\ts_nop 3"] + load)) == 1


@pytest.fixture(scope="module")
def code_objects(tmp_path_factory):
    from paper_2410_11720_amd import abft
    if OBJDUMP is None or READELF is None:
        pytest.skip("no disassembler")
    at = tmp_path_factory.mktemp("code")
    shutil.copy(abft.LIB_PATH, at / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", "lib.so"], cwd=at, check=True, capture_output=True)
    objs = [str(f) for f in at.iterdir() if "gfx950" in f.name and f.stat().st_size]
    assert objs
    return objs


def test_buffer_copies_wait_for_their_scalars(code_objects):
    copies, bad = 0, []
    for f in code_objects:
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", f], check=True,
                              capture_output=True, text=True).stdout.splitlines()
        copies += sum("buffer_load_dwordx4" in t and " lds" in t for t in text)
        bad += short_waits(text)
    assert copies > 0
    assert not bad, f"{len(bad)} short of {WAITS} wait states, first: {bad[:4]}"


def test_eight_wave_softmax_fits_twice(code_objects):
    seen = {}
    for f in code_objects:
        text = subprocess.run([READELF, "--notes", f], check=True, capture_output=True,
                              text=True).stdout
        for k in re.split(r"\n\s+- \.agpr_count:", text)[1:]:
            name = re.search(r"\.name:\s+(\S+)", k).group(1)
            if re.search(r"softmax_kernelI.*Li8ELb0EEEv", name):
                seen[name] = int(re.search(r"\.vgpr_count:\s+(\d+)", k).group(1))
    assert len(seen) == 16  # two types, one or two chunks, both directions, checked or not
    assert max(seen.values()) <= 128, {k: v for k, v in seen.items() if v > 128}
