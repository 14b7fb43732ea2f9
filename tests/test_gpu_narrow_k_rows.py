"""The staged kernel on k-rows shorter than a 16-byte chunk (a column-major A of a few rows, a row-major
B of a few columns): their loads reach over the rows behind them, so what is left of K after the
last whole step decides how many steps may be fetched that way.  And such operands keep the
prefetching: a product with four rows must not take longer than with twelve."""
import time

import pytest
import torch

import paper_2511_11939_amd as P
from test_gpu_parity import _general_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("la,lb,M,N", [("col", "row", 3, 140), ("col", "col", 1, 70), ("row", "row", 140, 2), ("col", "row", 7, 5)])
@pytest.mark.parametrize("ab", ["bf16", "f32"])
@pytest.mark.parametrize("K", [64, 65, 67, 71, 72, 97, 127, 129, 135, 193, 196, 513])
def test_short_k_rows(la, lb, M, N, ab, K):
    """Packed and padded rows: the padding holds values that would show in the result."""
    _general_case(M, N, K, ab=ab, la=la, lb=lb, ints=True)
    _general_case(M, N, K, ab=ab, la=la, lb=lb, pad=(1, 2, 1), offset=1, batch=2, ints=True)
    _general_case(M, N, K, ab=ab, la=la, lb=lb, split_k=2, ints=True)


def _time_us(M, N, K):
    A, B = (torch.randn(n, device="cuda").bfloat16() for n in (M * K, K * N))
    C, desc = torch.empty(M * N, device="cuda"), P.make_desc(c_dtype="f32", layout_a="col", layout_b="row", split_k=1)
    best = 1e9
    for _ in range(8):
        torch.cuda.synchronize()
        start = time.perf_counter()
        for _ in range(10):
            P.gemm(A, B, C, M=M, N=N, K=K, desc=desc)
        torch.cuda.synchronize()
        best = min(best, time.perf_counter() - start)
    return best * 1e5


def test_four_rows_take_no_longer_than_twelve():
    four, twelve = _time_us(4, 978, 10368), _time_us(12, 978, 10368)
    print(f"4 rows {four:.1f} us, 12 rows {twelve:.1f} us")
    assert four < 1.5 * twelve
