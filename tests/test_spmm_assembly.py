"""The tile kernels of tmask_spmm24 issue their matrix instructions from inline assembly, so the compiler does not know that
sums are in flight until the wait at the end of a tile's steps.  Here the compiled assembly is walked along its control
flow: between a matrix instruction and that wait nothing else may read or write an accumulation register (it would see
sums of up to eighteen wait states ago, without an error), and nothing but the direct copies may use m0, which they write."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2102_08124_amd import build

ACC = re.compile(r"\ba(\d+|\[\d+:\d+\])")


def _functions(text):
    """name -> instructions and labels, in order"""
    out, cur = {}, None
    for line in text.splitlines():
        line = line.split(";")[0].rstrip()
        m = re.match(r"(_Z\w+):", line)
        if m:
            cur = out.setdefault(m.group(1), [])
        elif line.startswith(".Lfunc_end"):
            cur = None
        elif cur is not None and (line.startswith(".LBB") or re.match(r"\s+[a-z]\w+", line)):
            cur.append(line.strip())
    return out


def _early_accesses(code):
    """Instructions that touch an accumulation register on some path from a matrix instruction to its wait."""
    label = {line[:-1]: i for i, line in enumerate(code) if line.endswith(":")}
    bad, seen, todo = set(), set(), [(0, False)]
    while todo:
        i, pending = todo.pop()
        if i >= len(code) or (i, pending) in seen:
            continue
        seen.add((i, pending))
        line = code[i]
        if line.startswith("v_smfmac"):
            pending = True
        elif line == "s_nop 15" and i + 1 < len(code) and code[i + 1] == "s_nop 15":
            pending = False
        elif pending and ACC.search(line):
            bad.add(line)
        if line.startswith("s_endpgm"):
            continue
        if "branch" in line:
            todo.append((label[line.split()[-1]], pending))
            if line.startswith("s_branch"):
                continue
        todo.append((i + 1, pending))
    return bad


def test_the_walk_finds_an_access_in_front_of_the_wait():
    loop = [".LBB0_1:", "v_smfmac_f32_32x32x32_bf16 a[0:15], v[0:3], v[4:11], v12", "s_cbranch_scc1 .LBB0_1"]
    store = ["global_store_dwordx4 v[0:1], a[0:3], off", "s_endpgm"]
    wait = ["s_nop 15", "s_nop 15"]
    assert _early_accesses(["v_accvgpr_write_b32 a0, 0"] + loop + wait + store) == set()
    assert _early_accesses(loop + ["v_accvgpr_mov_b32 a16, a0"] + wait + store) == {"v_accvgpr_mov_b32 a16, a0"}
    assert _early_accesses(loop + ["s_nop 15"] + store) == {store[0]}
    assert _early_accesses(loop + ["s_branch .LBB0_3", ".LBB0_2:"] + wait + [".LBB0_3:"] + store) == {store[0]}


def test_nothing_touches_the_sums_before_the_wait(tmp_path):
    if not (os.path.exists(build.HIPCC) or shutil.which(build.HIPCC)):
        pytest.skip("no hipcc")
    out = tmp_path / "spmm.s"
    flags = [f for f in build.FLAGS if f not in ("-shared", "-fPIC")]
    subprocess.run([build.HIPCC] + flags + ["--cuda-device-only", "-S", "-o", str(out), os.path.join(build.CSRC, "tmask_spmm.hip")],
                   check=True, capture_output=True)
    kernels = _functions(out.read_text())
    tile = {k: v for k, v in kernels.items() if "spmm24_tile_kernel" in k}
    assert len(tile) == 6
    for name, code in tile.items():
        assert sum(line.startswith("v_smfmac") for line in code) >= 8, name
        assert any(ACC.search(line) and "store" in line or "v_accvgpr_read" in line for line in code), name
        assert _early_accesses(code) == set(), name
    for name, code in kernels.items():
        copies = sum(line.startswith("global_load_lds") for line in code)
        assert sum(re.search(r"\bm0\b", line) is not None for line in code) == copies, name
