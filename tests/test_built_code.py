"""The machine code of the built library: spills where the compiler must not put them.

Where lanes come together again after a branch, a block begins with the instruction that
restores the lanes (s_or_b64 exec, exec, ..).  hipcc (ROCm 7.2) can put the store of a spilled
vector register ahead of it: only the lanes of the branch are saved, the others read back
whatever the slot held, and the results are wrong now and then, by what ran before.  A register
that the block itself has written is its own business."""

import os
import re
import shutil
import subprocess

import pytest

from paper_2407_14843_amd import build

OBJDUMP = next((p for p in ("/opt/rocm/llvm/bin/llvm-objdump", shutil.which("llvm-objdump") or "")
                if os.path.exists(p)), None)
WRITES = re.compile(r"v_|ds_read|ds_\w*_rtn|ds_bpermute|scratch_load|global_load|flat_load|buffer_load")


def registers(text):
    found = {(kind, int(n)) for kind, n in re.findall(r"\b([va])(\d+)\b", text)}
    for kind, lo, hi in re.findall(r"\b([va])\[(\d+):(\d+)\]", text):
        found |= {(kind, n) for n in range(int(lo), int(hi) + 1)}
    return found


def early_spills(lines):
    """(function, instruction) of every store of registers to scratch memory between a block's
    start and the restore of exec, of none of which the block has written a part."""
    found, function, block = [], "", None
    for line in lines:
        label = re.match(r"[0-9a-f]+ <(\w+)>:", line)
        if label:
            function = label.group(1) if label.group(1).startswith("_Z") else function
            block = []
            continue
        text = line.split("//")[0].strip()
        op = text.split(" ")[0]
        if block is None or not text:
            continue
        if op == "s_or_b64" and text.split()[1].startswith("exec"):
            written = set()
            for x in block:
                if x.startswith("scratch_store") and not registers(x) & written:
                    found.append((function, x))
                if WRITES.match(x):
                    written |= registers(x.split(",")[0])
            block = None
        elif op.startswith(("s_cbranch", "s_branch", "s_swappc", "s_setpc", "s_endpgm")) or (
                op.startswith("s_") and "exec" in text):
            block = None
        else:
            block.append(text)
    return found


def test_the_pattern_is_found():
    """The store that the compiler put wrong, as it was, and two that are in place."""
    body = ["000000000007fa34 <L4555>:", "\ts_mov_b32 s68, s34  // 0: 0", "{}",
            "\ts_or_b64 exec, exec, s[4:5]  // 0: 0"]
    wrong = "\tscratch_store_dword off, v18, s33 offset:68  // 0: 0"
    assert early_spills(x.format(wrong) for x in body) == [("", wrong.split("//")[0].strip())]
    own = ["\tv_add_u32_e32 v18, v1, v2", wrong]
    assert not early_spills(body[:2] + own + body[3:])
    assert not early_spills(body[:2] + body[3:] + [wrong])


@pytest.mark.skipif(OBJDUMP is None, reason="no llvm-objdump")
def test_no_spill_ahead_of_the_restore(tmp_path):
    shutil.copy(build.LIB_PATH, tmp_path / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", "lib.so"], cwd=tmp_path, check=True, capture_output=True)
    objects = [f for f in os.listdir(tmp_path) if "gfx950" in f]
    assert len(objects) == len(build.SOURCES), objects
    for f in objects:
        out = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", "--symbolize-operands", f],
                             cwd=tmp_path, check=True, capture_output=True, text=True).stdout
        assert not early_spills(out.splitlines())
