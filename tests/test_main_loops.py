"""The main loops of the built tile kernels, read in their own gfx950 assembly."""
import os
import re
import subprocess

import pytest

from paper_2604_24013_amd import build

LLVM = "/opt/rocm/llvm/bin"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{template arguments: [instructions and labels]} of gemm_bf16_dl_kernel"""
    d = str(tmp_path_factory.mktemp("dis"))
    obj = os.path.join(build.CSRC, "gemm_bf16_dl.o")
    if not os.path.exists(obj):
        build.build()
    run = lambda *a: subprocess.run(a, check=True, capture_output=True, text=True).stdout
    run(f"{LLVM}/llvm-objcopy", "--dump-section", f".hip_fatbin={d}/fat", obj, f"{d}/obj")
    run(f"{LLVM}/clang-offload-bundler", "--unbundle", "--type=o", "--targets=hipv4-amdgcn-amd-amdhsa--gfx950", f"--input={d}/fat",
        f"--output={d}/co")
    out, cur = {}, None
    for line in run(f"{LLVM}/llvm-objdump", "-d", "--symbolize-operands", "--no-show-raw-insn", f"{d}/co").splitlines():
        name = re.match(r"[0-9a-f]+ <(\w+)>:", line)
        if name and "gemm_bf16_dl_kernel" in name[1]:
            args = re.findall(r"L[ib](\d+)E", name[1])
            cur = out.setdefault(", ".join(args), [])
        elif name and name[1].startswith("L"):
            cur.append(name[1] + ":")
        elif name:
            cur = None
        elif cur is not None and line.startswith("\t"):
            cur.append(line.split("//")[0].strip())
    return out


def steady_loops(code):
    """Innermost loops that request one whole k-tile and multiply another: 16 MFMAs and more, at most eight loads to LDS."""
    at = {l[:-1]: i for i, l in enumerate(code) if l.endswith(":")}
    for i, l in enumerate(code):
        to = re.match(r"s_c?branch\w* (\w+)$", l)
        if to and at.get(to[1], i) < i:
            body = code[at[to[1]]:i + 1]
            loads = sum(x.startswith("buffer_load") and x.endswith(" lds") for x in body)
            if 4 <= loads <= 8 and sum("v_mfma" in x for x in body) >= 16 and len(body) < 900:
                yield body


def test_main_loops_keep_loads_in_flight(kernels):
    """Tiles whose loads are spread over the MFMAs: no trip may wait until nothing is in flight.  (What a work item still holds
    in registers from its last path can make the compiler do so, on every trip.)"""
    spread = {k: v for k, v in kernels.items() if k.split(", ")[5] == "1"}
    assert len(spread) >= 60
    drained = [k for k, code in spread.items()
               if any(re.search(r"s_waitcnt.*vmcnt\(0\)", x) for body in steady_loops(code) for x in body)]
    assert all(list(steady_loops(code)) for code in spread.values())
    assert drained == []
