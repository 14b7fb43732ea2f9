"""Host-only: which products of few rows take the kernel without tiles.  Problems that one launch of it could
not take stay on tiles, and so do those that tiles and a split are predicted to be faster at."""
import os
import subprocess

import paper_2511_11939_amd as P
from paper_2511_11939_amd import build


def _plan(M, N, K, batch=1, **kw):
    s, plan = P.prism_gemm_plan(P.make_desc(**kw), M, N, K, None, K, M * K, None, K, K * N, None, N, M * N, batch)
    assert s == P.Status.OK
    return plan


def test_very_wide_and_very_many_problems_are_still_accepted():
    assert _plan(1, 1 << 25, 64).kernel == 4
    assert _plan(1, (1 << 31) - 128, 64).kernel == 2
    assert _plan(16, 16, 64, batch=1 << 21).kernel == 4
    assert _plan(16, 16, 64, batch=1 << 23).kernel != 4


def test_a_long_way_for_few_workgroups_is_split_whatever_the_alignment():
    for K in (16384, 16383, 59410):
        plan = _plan(54, 52, K)
        assert plan.kernel in (1, 2) and plan.split_k >= 8, K
    assert _plan(56, 584, 59, batch=125).kernel == 1          # many rounds of short loops
    for M, N, K in ((8, 15702, 2816), (6, 15232, 3072)):      # half the compute units, operands from memory
        assert _plan(M, N, K).kernel == 4
    assert _plan(54, 52, 2000).kernel == 4 and _plan(16, 4096, 4096).kernel == 4


def test_without_a_split_there_is_no_reason_for_tiles():
    assert _plan(64, 512, 16384).split_k > 1
    for M, N, K in ((64, 512, 16384), (16, 512, 65536), (54, 52, 59410)):
        assert _plan(M, N, K, split_k=1).kernel == 4


def test_a_shared_b_is_counted_once_before_it_is_read_as_a_stream(tmp_path):
    source = tmp_path / "rule.hip"
    source.write_text("""#include "launch.hpp"
using prism::few_rows_stream_b;
static_assert(!few_rows_stream_b(4096, 4096, 2, 64, 0), "one B of 33 MB for all problems stays in the caches");
static_assert(few_rows_stream_b(4096, 4096, 2, 64, 4096 * 4096) && few_rows_stream_b(16384, 16384, 2, 1, 0), "these do not fit");
static_assert(!few_rows_stream_b(4096, 4096, 2, 8, 4096 * 4096) && few_rows_stream_b(8192, 16384, 4, 9, 0), "at and beyond 256 MB");
""")
    r = subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "--offload-arch=gfx950", "-std=c++17", "-fsyntax-only",
                        "--cuda-host-only", "-I", build.CSRC, str(source)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr


def test_too_few_stamps_are_refused_not_sent_to_another_kernel():
    """The stamped call is the same launch as the plain one, or none."""
    desc, base = P.make_desc(), 1 << 40
    plan = _plan(16, 4096, 4096)
    args = (desc, 16, 4096, 4096, base, 4096, 0, base << 1, 4096, 0, base << 2, 4096, 0, 1, base << 3)
    assert plan.kernel == 4
    assert P.prism_gemm_batched_stamped(*args, plan.workgroups * P.STAMP_BYTES_PER_WORKGROUP - 8) == P.Status.WORKSPACE


def test_a_hook_that_names_no_tile_changes_nothing(set_hook):
    for value, kernel in (("0", 2), ("1", 2), ("2", 4), ("11", 4)):
        set_hook("PRISM_GEMM_CONFIG", value)
        assert _plan(16, 4096, 4096).kernel == kernel, value
