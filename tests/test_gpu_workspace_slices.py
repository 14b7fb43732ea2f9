"""A call whose pitches or pointers send it to another kernel than aligned operands of the same shape
still splits its sum with the workspace that prism_gemm_workspace_size names for the shape, and
with less than that as far as it goes.  Integers, so that every slice must be there exactly once."""
import re

import pytest
import torch

import paper_2511_11939_amd as P

pytestmark = pytest.mark.gpu


def _split(capfd, M, N, K, *, batch=1, la="row", lb="col", pad=0, offset=0, workspace=None):
    """Runs the product with ones and twos as operands; returns the kernel and slices of its log line."""
    lda, ldb = (K if la == "row" else M) + pad, (N if lb == "row" else K)
    sa, sb = (M if la == "row" else K) * lda, (K if lb == "row" else N) * ldb
    A = torch.ones(batch * sa + offset, dtype=torch.bfloat16, device="cuda")
    B = torch.full((batch * sb,), 2.0, dtype=torch.bfloat16, device="cuda")
    C = torch.full((batch * M * N,), -1.0, device="cuda")
    desc = P.make_desc(c_dtype="f32", layout_a=la, layout_b=lb)
    s, nbytes = P.prism_gemm_workspace_size(desc, M, N, K, batch)
    assert s == 0
    nbytes = nbytes if workspace is None else workspace
    ws = torch.full((nbytes + 64,), 0x5A, dtype=torch.uint8, device="cuda")
    desc.workspace, desc.workspace_bytes = ws.data_ptr(), nbytes
    capfd.readouterr()
    P.gemm(A.data_ptr() + 2 * offset, B, C, M=M, N=N, K=K, desc=desc, lda=lda, batch=batch, strideA=sa, strideB=sb, strideC=M * N)
    torch.cuda.synchronize()
    line = capfd.readouterr().err
    assert bool((C == 2.0 * K).all()) and bool((ws[nbytes:] == 0x5A).all())
    return re.search(r"kernel=(\w+)", line).group(1), int(re.search(r"split_k=(\d+)", line).group(1))


def test_unaligned_operands_use_the_queried_workspace(set_hook, capfd):
    set_hook("PRISM_LOG", "1")
    for M, N, K, la, lb, pad in ((256, 256, 32768, "col", "row", 0), (512, 256, 32768, "col", "row", 0), (1, 64, 13376, "col", "col", 8),
                                 (200, 300, 40960, "row", "col", 0)):
        kernel, split = _split(capfd, M, N, K, la=la, lb=lb, pad=pad, offset=1)
        assert kernel == "gemm_staged" and split >= 8, (M, N, K)


def test_rows_too_far_apart_for_the_kernel_for_few_rows(set_hook, capfd):
    set_hook("PRISM_LOG", "1")
    kernel, split = _split(capfd, 4, 512, 4096, pad=(1 << 21) - 4096)
    assert kernel == "gemm_staged" and split > 1


@pytest.mark.parametrize("slabs,most", [(0.5, 1), (1, 1), (2, 2), (3.9, 3), (7, 7), (1000, 1000)])
def test_a_smaller_workspace_holds_fewer_slices(slabs, most, set_hook, capfd):
    set_hook("PRISM_LOG", "1")
    _, split = _split(capfd, 136, 264, 8192, workspace=int(slabs * 136 * 264 * 4))
    assert split == 1 if most == 1 else 1 < split <= most


def test_without_room_for_a_split_few_rows_are_not_left_to_tiles(set_hook, capfd):
    set_hook("PRISM_LOG", "1")
    assert _split(capfd, 64, 512, 16384) == ("gemm_pipelined", 16)
    assert _split(capfd, 64, 512, 16384, workspace=0) == ("gemm_skinny", 1)
