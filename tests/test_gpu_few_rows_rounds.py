"""Few rows: one or two blocks of columns per workgroup, by how full the last round of workgroups is."""
import pytest

import paper_2511_11939_amd as P
from test_gpu_parity import _general_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,K,columns", [(16, 8192, 256, 32), (16, 8193, 256, 16), (5, 12300, 200, 32), (16, 16384, 128, 32), (16, 16390, 128, 16),
                                           (17, 8200, 256, 32), (33, 8200, 3072, 16)])
def test_columns_per_workgroup(M, N, K, columns):
    s, plan = P.prism_gemm_plan(P.make_desc(c_dtype="f32"), M, N, K, None, K, 0, None, K, 0, None, N, 0, 1)
    assert s == 0 and plan.kernel == 4 and plan.tile_n == columns and plan.workgroups == -(-N // columns)
    _general_case(M, N, K, ints=True)
