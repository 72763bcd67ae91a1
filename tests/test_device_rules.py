"""The plain arithmetic that the device code and the host share
(csrc/mce_internal.h), compiled for the host and run at the ends of its ranges."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    src, lib = str(d / "rules.cpp"), str(d / "rules.so")
    with open(src, "w") as f:
        f.write('#include "mce_internal.h"\nusing namespace mce;\n' + SOURCE)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__",
                           "-I/opt/rocm/include", "-I" + os.path.join(ROOT, "include"),
                           "-I" + os.path.join(ROOT, "paper_1801_00202_amd", "csrc"), "-o", lib, src])
    return ctypes.CDLL(lib)


SOURCE = r"""
// children, nodes and cliques of a lane search that holds `start` of each and
// takes `steps` more of 64 busy lanes, each a node, with 64 cliques a step
extern "C" void lane_totals(uint64_t start, uint32_t steps, uint64_t* out)
{
    LaneTotals t;
    t.children = t.nodes = t.cliques = start;
    for (uint32_t i = 0; i < steps; i++) {
        t.step(64, 64);
        t.cliques += 64;
    }
    out[0] = t.children;
    out[1] = t.nodes;
    out[2] = t.cliques;
}
"""


@pytest.mark.parametrize("start", [0, (1 << 32) - 65, (1 << 32) - 64, (1 << 32) - 1, 1 << 40])
def test_lane_totals_pass_32_bits(rules, start):
    out = (ctypes.c_uint64 * 3)()
    rules.lane_totals(ctypes.c_uint64(start), ctypes.c_uint32(3), out)
    assert list(out) == [start + 192] * 3
