"""The waits that the memory-to-LDS product kernels of csrc/linear.hip owe to their source alone.

Behind the barrier of a slab other wavefronts' loads overwrite the LDS stage it frees, and those keep no order with a fragment read
that is still under way: a wavefront has to wait for its reads (lgkmcnt) and for its part of the next slab (vmcnt) before it gets there.
Whether the compiled code happens to wait is up to the scheduler, so what is looked at is the device code before any optimisation."""
import os
import re
import subprocess

import pytest

from paper_2506_01206_amd import build

LIST = re.compile(r"@llvm\.amdgcn\.s\.waitcnt\(i32 (\d+)\)|call void @\S*(lds_barrier_linear)\S*\(")


@pytest.fixture(scope="module")
def functions(tmp_path_factory):
    """name -> the function's waits (their immediates) and barriers ("barrier"), in order"""
    out = tmp_path_factory.mktemp("ir") / "linear.ll"
    flags = [f for f in build.FLAGS if f not in ("-O3", "-fPIC", "-Wall")]
    flags = flags[:flags.index("-mllvm")] + flags[flags.index("-mllvm") + 2:]      # (an option of the code generator)
    subprocess.check_call([build.HIPCC] + flags + ["-O3", "--cuda-device-only", "-S", "-emit-llvm", "-Xclang", "-disable-llvm-passes", "-w",
                                                   os.path.join(build.CSRC, "linear.hip"), "-o", str(out)])
    found = {}
    for body in re.findall(r"^define [^\n]*\n.*?^}", out.read_text(), re.S | re.M):
        name = re.search(r'@"?([\w.$]+)"?\(', body).group(1)
        found[name] = [int(a) if a else "barrier" for a, b in LIST.findall(body.split("\n", 1)[1])]
    return found


def counters(imm):
    """vmcnt, lgkmcnt of an s_waitcnt immediate (63 and 15: not waited for)"""
    return (imm & 15) | (imm >> 14 & 3) << 4, imm >> 8 & 15


def test_a_stage_is_freed_only_when_its_fragments_are_in_registers(functions):
    slabs = {n: l for n, l in functions.items() if "linear_wide_kernel" in n and n.startswith("_ZZ") and "barrier" in l}
    assert len(slabs) >= 4 * 5                                     # four forms of a slab in every kind of tile
    for name, l in slabs.items():
        assert len(l) == 2 and l[1] == "barrier" and counters(l[0]) == (0, 0), (name, l)
    rings = {n: l for n, l in functions.items() if "linear_ring_kernel" in n and n.startswith("_ZN")}
    assert len(rings) >= 3
    for name, l in rings.items():                                  # (the loads of the next slab: by count, in a function of their own)
        assert l[:3] == ["barrier", l[1], "barrier"] and counters(l[1])[1] == 0, (name, l)
