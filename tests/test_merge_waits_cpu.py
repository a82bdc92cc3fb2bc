"""The streaming merge (csrc/merge_mfma.hpp, merge_mid_rows) waits for all but its newest memory operations, a number that
counts what a stage issues.  That number is right only while the compiler issues exactly those, and the stores write the
right values only while their offset within the stage is in a vector register.  Here both are read off the built library."""
import collections
import re
import subprocess

import pytest

from paper_2605_00392_amd import build

LLVM = "/opt/rocm/llvm/bin/"
PIECES = 8                                             # a stage's loads and stores of kept rows by a lane (kPieces)


@pytest.fixture(scope="module")
def code(tmp_path_factory):
    path = tmp_path_factory.mktemp("code")
    run = lambda *a: subprocess.run(a, check=True, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True).stdout
    run(LLVM + "llvm-objcopy", f"--dump-section=.hip_fatbin={path}/bundle", build.LIB_PATH, f"{path}/unused")
    run(LLVM + "clang-offload-bundler", "--unbundle", "--type=o", "--targets=hipv4-amdgcn-amd-amdhsa--gfx950",
        f"--input={path}/bundle", f"--output={path}/device")
    text = run(LLVM + "llvm-objdump", "-d", "--mcpu=gfx950", f"{path}/device")
    functions = re.split(r"\n[0-9a-f]+ <", text)
    return next(f for f in functions if f.startswith("_ZN3rtp13k_merge_lists")).splitlines()


KINDS = (("load", r"\bbuffer_load_dwordx4\b"), ("lds", r"\bglobal_load_lds_dwordx4\b"), ("store", r"\bbuffer_store_dwordx4\b"))


def operation(line):
    """0, 1, 2: a memory operation of a stage; None: none."""
    return next((k for k, (_, pattern) in enumerate(KINDS) if re.search(pattern, line)), None)


def paths_from(code, start, stop):
    """Every (place, operations by kind) at which a path from line `start` meets a line in `stop` or the end."""
    address = lambda line: int(re.search(r"// ([0-9A-F]+):", line).group(1), 16)
    lines = {address(line): i for i, line in enumerate(code) if re.search(r"// [0-9A-F]+:", line)}
    base = min(lines)
    target = lambda line: lines[base + int((re.search(r"<.*\+0x([0-9a-f]+)>", line) or re.match("()", "")).group(1) or "0", 16)]
    seen, ends, todo = set(), set(), [(start + 1, (0, 0, 0))]
    while todo:
        i, count = todo.pop()
        if (i, count) in seen or max(count) > 4 * PIECES:
            assert max(count) <= 4 * PIECES, i
            continue
        seen.add((i, count))
        line = code[i]
        if i in stop or "s_endpgm" in line:
            ends.add((i, count))
            continue
        k = operation(line)
        if k is not None:
            count = tuple(c + (j == k) for j, c in enumerate(count))
        if "s_branch" in line or "s_cbranch" in line:
            todo.append((target(line), count))
        if "s_branch" not in line:
            todo.append((i + 1, count))
    return ends


@pytest.mark.parametrize("blocks", [1, 2])
def test_the_counted_waits_count_what_is_issued(code, blocks):
    """`blocks` of 32 pruned rows: 2 of their requests a wave and stage each, straight into LDS."""
    requests = 2 * blocks
    full, last = 3 * PIECES + requests, 2 * PIECES
    is_full = lambda line: re.search(rf"s_waitcnt vmcnt\({full}\) lgkmcnt\(0\)", line)
    counted = {i for i, line in enumerate(code) if is_full(line) or re.search(rf"s_waitcnt vmcnt\(({last}|0)\) lgkmcnt\(0\)", line)}
    # (a stage's wait is for one of two numbers, each behind a branch of its own: a path that takes neither, which there is
    # none of, ends there too)
    stop = counted | {i - k for i in counted for k in (1, 2) if "s_cbranch" in code[i - k]}
    waits = [i for i, line in enumerate(code) if is_full(line)]
    assert len(waits) >= 5, len(waits)                 # three stages of the long loop, one to four that are left
    # what is in flight at the first: two stages' requests, and stores that stand for those of two stages before
    first = [operation(line) for line in code[:waits[0]]]
    first = collections.Counter([k for k in first if k is not None][-2 * (2 * PIECES + requests):])
    assert first == {0: 2 * PIECES, 1: 2 * requests, 2: 2 * PIECES}, first
    requested = 0
    for wait in waits:                                 # from a stage's wait to the next stage's
        ends = paths_from(code, wait, stop)
        assert ends
        for i, (loads, lds, stores) in ends:
            assert stores == PIECES and (loads, lds) in ((PIECES, requests), (0, 0)), (wait, i, loads, lds, stores)
            requested += loads > 0
    assert requested >= 3


def test_no_store_has_a_scalar_offset(code):
    stores = [line for line in code if re.search(r"\bbuffer_store_dwordx4\b", line)]
    assert stores and all(re.search(r"buffer_store_dwordx4 v\[\d+:\d+\], v\d+, s\[\d+:\d+\], 0 offen", line) for line in stores)


def test_nothing_of_the_kernel_is_spilled(code):
    """(A spilled register's load or store would be one more memory operation.)"""
    assert not [line for line in code if "scratch_" in line]
