"""The kernel for few rows where it can go wrong: rows around its block sizes, columns around a
block and around the line between one and two blocks per workgroup, K shorter than a chunk's
neighbourhood, K that leaves waves without a step, partial last steps, unaligned rows."""
import pytest
import torch

import paper_2511_11939_amd as P
from test_gpu_parity import _general_case

pytestmark = pytest.mark.gpu


def _plan(M, N, K, ab="bf16", batch=1, **kw):
    desc = P.make_desc(ab_dtype=ab, c_dtype="f32", **kw)
    s, plan = P.prism_gemm_plan(desc, M, N, K, None, K, M * K, None, K, K * N, None, N, M * N, batch)
    assert s == 0
    return plan


@pytest.mark.parametrize("M", [1, 5, 16, 17, 32, 33, 64])
@pytest.mark.parametrize("N,K", [(1, 64), (15, 8), (16, 72), (17, 512), (100, 1000), (40, 2048), (8200, 200), (33, 4160), (64, 65)])
def test_rows_columns_and_k(M, N, K):
    assert _plan(M, N, K).kernel == 4
    _general_case(M, N, K, ints=True)
    _general_case(M, N, K, ab="f16", cd="f16", bias=True, alpha=-0.5, beta=0.25, pad=(1, 3, 1))


@pytest.mark.parametrize("M,N,K", [(3, 50, 4), (16, 33, 37), (20, 300, 1024), (64, 8200, 65), (40, 17, 5)])
def test_fp32_operands(M, N, K):
    assert _plan(M, N, K, ab="f32").kernel == 4
    _general_case(M, N, K, ab="f32", ints=True)
    _general_case(M, N, K, ab="f32", alpha=1.5, beta=0.5, bias=True, pad=(1, 1, 1), offset=1)


def test_batches_column_major_results_and_the_rule():
    _general_case(9, 50, 130, batch=7, pad=(2, 1, 3), bias=True)
    _general_case(300, 9, 130, lc="col", bias=True, cd="bf16")       # runs as C^T with nine rows
    _general_case(16, 272, 96, batch=64, ints=True)
    assert _plan(64, 512, 512).kernel == 4 and _plan(65, 512, 512).kernel != 4
    assert _plan(16, 512, 7).kernel != 4                             # shorter than a chunk
    assert _plan(16, 512, 512, layout_b="row").kernel != 4
    assert _plan(16, 512, 512, split_k=2).kernel != 4
    assert _plan(64, 16384, 4096).kernel == 2 and _plan(32, 16384, 4096).kernel == 4      # tiles enough for the chip
    assert _plan(64, 512, 16384).kernel == 2 and _plan(64, 512, 4096).kernel == 4         # a long way for few workgroups
    assert _plan(16, 8191, 512).tile_n == 32 and _plan(16, 8160, 512).tile_n == 16


def test_stamped_launch_and_repeated_results():
    a = torch.randn(16, 2048, device="cuda").bfloat16()
    b = torch.randn(4096, 2048, device="cuda").bfloat16()
    out = [torch.empty(16, 4096, dtype=torch.bfloat16, device="cuda") for _ in range(3)]
    desc = P.make_desc()
    plan = _plan(16, 4096, 2048)
    for c in out[:2]:
        P.gemm(a, b, c, M=16, N=4096, K=2048, desc=desc)
    stamps = torch.zeros(plan.workgroups * 8, dtype=torch.int64, device="cuda")
    assert P.prism_gemm_batched_stamped(desc, 16, 4096, 2048, a, 2048, 0, b, 2048, 0, out[2], 4096, 0, 1, stamps,
                                        stamps.numel() * 8, torch.cuda.current_stream().cuda_stream) == 0
    torch.cuda.synchronize()
    assert torch.equal(out[0], out[1]) and torch.equal(out[0], out[2])
    assert (stamps.view(-1, 4, 2)[:, :, 0].diff(dim=1) > 0).all()
