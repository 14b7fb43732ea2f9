"""Race check in every layout: the library built with full barriers (and, inside a wave, full waits) after
every LDS phase gives the same bits as the normal build for the 256x256 tiles with k-rows, for
staged loops long enough that two K steps travel in registers while two lie in LDS, and for the
kernel for few rows, whose waves pass every step through LDS of their own."""
import ctypes

import pytest
import torch

import paper_2511_11939_amd as P
from test_gpu_paranoid_barriers import paranoid  # noqa: F401

pytestmark = pytest.mark.gpu
LAYOUTS = [("row", "col"), ("row", "row"), ("col", "col"), ("col", "row")]
TYPES = {"bf16": torch.bfloat16, "f16": torch.float16, "f32": torch.float32}


def _same_bits(paranoid, set_hook, M, N, K, kernel, la="row", lb="col", ab="bf16", hooks=(), tile_m=None):
    for name, value in dict(hooks).items():
        set_hook(name, value)
    paranoid.prism_reread_environment()
    lda, ldb = (K if la == "row" else M), (N if lb == "row" else K)
    desc = P.make_desc(ab_dtype=ab, c_dtype="f32", layout_a=la, layout_b=lb, split_k=1)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(M + N + K)
    A, B = (torch.randn(n, device="cuda", generator=gen).to(TYPES[ab]) for n in (M * K, K * N))
    s, plan = P.prism_gemm_plan(desc, M, N, K, A, lda, 0, B, ldb, 0, None, N, 0, 1)
    assert s == 0 and plan.kernel == kernel and tile_m in (None, plan.tile_m)
    outs = []
    for lib in (P.load_library(), paranoid):
        C = torch.full((M * N,), float("nan"), device="cuda")
        assert lib.prism_gemm_batched(ctypes.byref(desc), M, N, K, A.data_ptr(), lda, 0, B.data_ptr(), ldb, 0, C.data_ptr(), N, 0, 1,
                                      torch.cuda.current_stream().cuda_stream) == 0
        torch.cuda.synchronize()
        outs.append(C)
    assert not outs[0].isnan().any()
    assert torch.equal(outs[0].view(torch.int32), outs[1].view(torch.int32))


@pytest.fixture(autouse=True)
def _hooks_restored(request):
    yield
    if "paranoid" in request.fixturenames:      # it keeps its own copy of the hooks
        import os
        os.environ.pop("PRISM_GEMM_CONFIG", None)
        request.getfixturevalue("paranoid").prism_reread_environment()


@pytest.mark.parametrize("la,lb", LAYOUTS[1:])
@pytest.mark.parametrize("ksteps", [1, 2, 5, 8])
def test_large_tiles_with_k_rows(paranoid, set_hook, la, lb, ksteps):  # noqa: F811
    _same_bits(paranoid, set_hook, 776, 520, 64 * ksteps, 2, la, lb, hooks={"PRISM_GEMM_CONFIG": "0"}, tile_m=256)


@pytest.mark.parametrize("la,lb", LAYOUTS)
@pytest.mark.parametrize("ab,K", [("bf16", 323), ("f16", 451), ("f32", 161), ("f32", 250)])
def test_staged_loops_of_five_to_eight_steps(paranoid, set_hook, la, lb, ab, K):  # noqa: F811
    _same_bits(paranoid, set_hook, 300, 203, K, 1, la, lb, ab)


@pytest.mark.parametrize("M,N,K,ab", [(1, 4096, 4096, "bf16"), (16, 517, 2088, "f16"), (33, 3000, 1000, "bf16"), (64, 8200, 200, "bf16"),
                                      (20, 300, 1024, "f32"), (64, 8200, 65, "f32")])
def test_few_rows(paranoid, set_hook, M, N, K, ab):  # noqa: F811
    _same_bits(paranoid, set_hook, M, N, K, 4, ab=ab)
