"""The norm pass on tokens wider than 1280 (csrc/stage1.hpp, k_norms) runs a wave or two to a SIMD: a row's sixteen loads have to be in
flight together.  Read off the built library: no wait for memory between the first and the last of them."""
import re
import subprocess

import pytest

from paper_2605_00392_amd import build

LLVM = "/opt/rocm/llvm/bin/"


@pytest.fixture(scope="module")
def functions(tmp_path_factory):
    path = tmp_path_factory.mktemp("code")
    run = lambda *a: subprocess.run(a, check=True, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True).stdout
    run(LLVM + "llvm-objcopy", f"--dump-section=.hip_fatbin={path}/bundle", build.LIB_PATH, f"{path}/unused")
    run(LLVM + "clang-offload-bundler", "--unbundle", "--type=o", "--targets=hipv4-amdgcn-amd-amdhsa--gfx950",
        f"--input={path}/bundle", f"--output={path}/device")
    return re.split(r"\n[0-9a-f]+ <", run(LLVM + "llvm-objdump", "-d", "--mcpu=gfx950", f"{path}/device"))


@pytest.mark.parametrize("variance", [0, 1])
@pytest.mark.parametrize("dtype, load", [("t", "global_load_dwordx2"), ("f", "global_load_dwordx4")])
def test_a_rows_loads_are_in_flight_together(functions, dtype, load, variance):
    code = next(f for f in functions if f.startswith(f"_ZN3rtp7k_normsI{dtype}Li16ELi0ELb{variance}E")).splitlines()
    loads = [i for i, line in enumerate(code) if re.search(rf"\b{load}\b.*\bnt\b", line)]
    assert len(loads) == 16, len(loads)
    between = code[loads[0]:loads[-1]]
    assert not [line for line in between if "vmcnt" in line or "s_cbranch" in line or "s_branch" in line]
