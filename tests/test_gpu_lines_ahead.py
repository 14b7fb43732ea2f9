"""Large tiles whose operands come from memory ask for a K step's lines before its copies: K loops of one to
seven steps, edges in both directions, slices.  Integers, exact against torch in fp32, and the
race-check build gives the same bits."""
import ctypes
import os

import pytest
import torch

import paper_2511_11939_amd as P
from test_gpu_paranoid_barriers import paranoid  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _hooks_restored(paranoid):  # noqa: F811
    yield
    for name in ("PRISM_GEMM_CONFIG", "PRISM_PERSISTENT"):
        os.environ.pop(name, None)
    paranoid.prism_reread_environment()         # it keeps its own copy of the hooks


@pytest.mark.parametrize("la,lb,M,N,K", [
    ("row", "col", 840008, 264, 64), ("row", "col", 420009, 259, 128), ("row", "col", 280003, 140, 192), ("row", "col", 120007, 520, 448),
    ("row", "col", 777, 1033, 32832), ("row", "row", 170003, 264, 320), ("col", "col", 170008, 261, 320),
    ("col", "row", 100008, 264, 320), ("col", "row", 33000, 776, 1024), ("col", "row", 1000, 776, 32832)])
def test_exact_and_the_same_bits_as_the_race_check_build(paranoid, set_hook, la, lb, M, N, K):  # noqa: F811
    set_hook("PRISM_GEMM_CONFIG", "0")
    set_hook("PRISM_PERSISTENT", "0")
    paranoid.prism_reread_environment()
    gen = torch.Generator(device="cuda")
    gen.manual_seed(M + N + K)
    A, B = (torch.randint(-8, 9, s, device="cuda", generator=gen).float() for s in ((M, K), (K, N)))
    want = A @ B
    a, b = (A if la == "row" else A.t().contiguous()).bfloat16(), (B if lb == "row" else B.t().contiguous()).bfloat16()
    del A, B
    desc = P.make_desc(c_dtype="f32", layout_a=la, layout_b=lb)
    s, nbytes = P.prism_gemm_workspace_size(desc, M, N, K, 1)
    ws = torch.empty(max(nbytes, 1), dtype=torch.uint8, device="cuda")
    desc.workspace, desc.workspace_bytes = ws.data_ptr(), nbytes
    lda, ldb = (K if la == "row" else M), (N if lb == "row" else K)
    s, plan = P.prism_gemm_plan(desc, M, N, K, a, lda, 0, b, ldb, 0, None, N, 0, 1)
    assert s == 0 and plan.kernel == 2 and plan.tile_m == 256 and 2 * K * (M + N) > 6.0e7
    for lib in (P.load_library(), paranoid):
        C = torch.full((M, N), float("nan"), device="cuda")
        assert lib.prism_gemm_batched(ctypes.byref(desc), M, N, K, a.data_ptr(), lda, 0, b.data_ptr(), ldb, 0, C.data_ptr(), N, 0, 1,
                                      torch.cuda.current_stream().cuda_stream) == 0
        torch.cuda.synchronize()
        assert torch.equal(C, want)
