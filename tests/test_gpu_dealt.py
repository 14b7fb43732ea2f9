"""The kernel whose workgroups deal K steps to their waves, where it can go wrong: sizes around its workgroups
(32 x 32, 128 x 64), waves without a step, K that ends inside a step, a chunk and an element,
rows that start in the middle of a 32-bit word (also a problem's or a slice's first), k-rows whose
loads would run past the operand's end, and slices.  Integers must come out exactly; the padding
around the operands holds values that would show.  The race-check build gives the same bits."""
import ctypes

import pytest
import torch

import paper_2511_11939_amd as P
from test_gpu_paranoid_barriers import paranoid  # noqa: F401
from test_gpu_parity import _general_case

pytestmark = pytest.mark.gpu
LAYOUTS = [("row", "col"), ("row", "row"), ("col", "col"), ("col", "row")]
TYPES = {"bf16": torch.bfloat16, "f32": torch.float32}


def _plan(M, N, K, la="row", lb="col", ab="bf16", batch=1, **kw):
    desc = P.make_desc(ab_dtype=ab, c_dtype="f32", layout_a=la, layout_b=lb, **kw)
    s, plan = P.prism_gemm_plan(desc, M, N, K, None, K if la == "row" else M, M * K, None, N if lb == "row" else K, K * N, None, N, M * N, batch)
    assert s == 0
    return plan


def _dealt(plan):
    return plan.kernel in (1, 2) and plan.tile_n < 128


@pytest.mark.parametrize("la,lb", LAYOUTS)
@pytest.mark.parametrize("ab", ["bf16", "f32"])
@pytest.mark.parametrize("M,N,K", [(65, 1, 64), (66, 33, 65), (97, 31, 191), (128, 65, 33), (127, 64, 512), (96, 96, 1100), (161, 40, 1027)])
def test_sizes_and_layouts(la, lb, ab, M, N, K):
    if N > 8 and K > 64:
        assert _dealt(_plan(M, N, K, la, lb, ab))
    _general_case(M, N, K, ab=ab, la=la, lb=lb, ints=True)
    _general_case(M, N, K, ab=ab, la=la, lb=lb, pad=(1, 3, 1), batch=3, ints=True)         # odd rows and odd problems
    _general_case(M, N, K, ab=ab, la=la, lb=lb, lc="col", pad=(2, 2, 3), offset=1, bias=True, alpha=-0.5, beta=0.25)


@pytest.mark.parametrize("la,lb", LAYOUTS)
@pytest.mark.parametrize("M,N,K", [(1030, 900, 700), (1025, 1057, 301)])
def test_workgroups_of_128_rows(la, lb, M, N, K):
    _general_case(M, N, K, la=la, lb=lb, ab="f16", cd="f16", ints=True)


@pytest.mark.parametrize("la,lb", LAYOUTS)
@pytest.mark.parametrize("M,N,K", [(70, 50, 9000), (97, 33, 8963)])
def test_slices(la, lb, M, N, K):
    plan = _plan(M, N, K, la, lb)
    assert _dealt(plan) and plan.split_k > 1 and plan.workspace_bytes == plan.split_k * M * N * 4
    _general_case(M, N, K, la=la, lb=lb, ints=True)
    assert _plan(M, N, K, la, lb, split_k=1).split_k == 1


def test_the_hook_keeps_tiles(set_hook):
    assert _dealt(_plan(300, 200, 323)) and _dealt(_plan(304, 200, 320))
    set_hook("PRISM_GEMM_CONFIG", "1")
    assert not _dealt(_plan(300, 200, 323)) and not _dealt(_plan(304, 200, 320))


@pytest.mark.parametrize("la,lb", LAYOUTS)
@pytest.mark.parametrize("ab", ["bf16", "f32"])
@pytest.mark.parametrize("K", [101, 160, 327])
def test_staged_tiles_still_serve_these_sizes(la, lb, ab, K, set_hook):
    set_hook("PRISM_GEMM_CONFIG", "1")
    _general_case(131, 139, K, ab=ab, la=la, lb=lb, pad=(1, 3, 1), ints=True)
    _general_case(5, 139, K, ab=ab, la=la, lb=lb, batch=2, offset=1, ints=True)


@pytest.mark.parametrize("la,lb", LAYOUTS)
@pytest.mark.parametrize("ab,M,N,K", [("bf16", 193, 77, 1003), ("bf16", 192, 80, 1024), ("f32", 193, 77, 500), ("bf16", 1200, 1000, 501)])
def test_race_check_build(paranoid, la, lb, ab, M, N, K):  # noqa: F811
    desc = P.make_desc(ab_dtype=ab, c_dtype="f32", layout_a=la, layout_b=lb, split_k=1)
    A, B = (torch.randn(n, device="cuda").to(TYPES[ab]) for n in (M * K, K * N))
    outs = []
    for lib in (P.load_library(), paranoid):
        C = torch.full((M * N,), float("nan"), device="cuda")
        assert lib.prism_gemm_batched(ctypes.byref(desc), M, N, K, A.data_ptr(), K if la == "row" else M, 0, B.data_ptr(),
                                      N if lb == "row" else K, 0, C.data_ptr(), N, 0, 1, torch.cuda.current_stream().cuda_stream) == 0
        torch.cuda.synchronize()
        outs.append(C)
    assert not outs[0].isnan().any() and torch.equal(outs[0].view(torch.int32), outs[1].view(torch.int32))


@pytest.mark.parametrize("la,lb", LAYOUTS)
@pytest.mark.parametrize("M,N,K", [(960, 904, 1088), (961, 903, 1087)])
def test_workgroups_of_64_rows(la, lb, M, N, K):
    plan = _plan(M, N, K, la, lb)
    assert _dealt(plan) and plan.tile_n == 64 and plan.workgroups == -(-M // 64) * -(-N // 64)
    _general_case(M, N, K, la=la, lb=lb, ab="f16", cd="f16", ints=True)
    _general_case(M, N, K, la=la, lb=lb, lc="col", pad=(1, 1, 3), bias=True, alpha=-0.5, beta=0.25)
