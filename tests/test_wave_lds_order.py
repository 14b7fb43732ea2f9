"""Lanes of one wave that pass values to each other through LDS: to the compiler a lane's reads of what
others wrote look unrelated to its own writes.  A value read before the write must be read again
after it.  Device code of a small kernel, compiled here; no GPU needed."""
import os
import re
import subprocess

from paper_2511_11939_amd import build

SOURCE = """#include "wave.hpp"
using namespace prism;
extern "C" __global__ void passes(int* out)
{
    __shared__ int lds[65];
    const persp::Wave wv = persp::Grid::at_kernel_entry().workgroup<64>().wave();
    const int lane = threadIdx.x & 63, reader = lane + %s;
    const int before = lds[reader + 1];
    lds[lane] = lane;
    out[lane] = lds[reader + 1];
    out[64 + lane] = before;
}
"""


def _lds_accesses(tmp_path, reader):
    source, asm = tmp_path / "passes.hip", tmp_path / "passes.s"
    source.write_text(SOURCE % reader)
    r = subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "--offload-arch=gfx950", "-O3", "-std=c++17", "-S",
                        "--cuda-device-only", "-I", build.CSRC, str(source), "-o", str(asm)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return re.findall(r"^\s+ds_(read|write)", asm.read_text(), re.M)


def test_a_wave_reads_again_what_other_lanes_have_written(tmp_path):
    assert _lds_accesses(tmp_path, "wave::unknown_offset(wv)") == ["read", "write", "read"]


def test_the_kernels_that_pass_values_this_way_say_so():
    """The kernel for few rows and the epilogue's patch; both units are in the race-check build."""
    for unit, waits in (("skinny.hip", 3), ("workgroup.hpp", 2)):
        source = open(os.path.join(build.CSRC, unit)).read()
        assert source.count("wave::unknown_offset(wv)") == 1 and source.count("PRISM_PARANOID_WAIT()") == waits, unit
    assert {"kernels.hip", "skinny.hip"} <= set(build._PARANOID_UNITS)
