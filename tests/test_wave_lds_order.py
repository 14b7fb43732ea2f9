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
    const int lane = threadIdx.x & 63;
    const int before = lds[lane + 1];
    %s;
    lds[lane] = lane;
    %s;
    out[lane] = lds[lane + 1];
    out[64 + lane] = before;
}
"""


def _lds_accesses(tmp_path, between):
    source, asm = tmp_path / "passes.hip", tmp_path / "passes.s"
    source.write_text(SOURCE % (between, between))
    r = subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "--offload-arch=gfx950", "-O3", "-std=c++17", "-S",
                        "--cuda-device-only", "-I", build.CSRC, str(source), "-o", str(asm)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return re.findall(r"^\s+ds_(read|write)", asm.read_text(), re.M)


def test_a_wave_reads_again_what_other_lanes_have_written(tmp_path):
    assert _lds_accesses(tmp_path, "wave::lds_in_order(wv)") == ["read", "write", "read"]


def test_the_kernels_that_pass_values_this_way_say_so():
    """The kernel for few rows (a step, and the reads before the next step) and the epilogue's patch."""
    assert open(os.path.join(build.CSRC, "skinny.hip")).read().count("wave::lds_in_order(wv)") == 2
    assert open(os.path.join(build.CSRC, "workgroup.hpp")).read().count("wave::lds_in_order(wv)") == 2
    assert {"kernels.hip", "skinny.hip"} <= set(build._PARANOID_UNITS)
