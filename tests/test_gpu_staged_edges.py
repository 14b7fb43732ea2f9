"""The staged kernel where it can go wrong: K around whole and partial steps and chunks, rows and
columns around chunks and tiles, dimensions shorter than a chunk, in every layout pair and every
element size.  Integers must come out exactly; the padding around the operands holds values that
would show in the result if an element beyond the matrix were used."""
import pytest

import paper_2511_11939_amd as P
from test_gpu_parity import _general_case

pytestmark = pytest.mark.gpu

LAYOUTS = [("row", "col"), ("row", "row"), ("col", "col"), ("col", "row")]


@pytest.mark.parametrize("la,lb", LAYOUTS)
@pytest.mark.parametrize("ab", ["bf16", "f32"])
@pytest.mark.parametrize("K", [1, 5, 8, 31, 33, 63, 65, 129, 191, 257, 323])
def test_k_tails(la, lb, ab, K):
    """One to eleven K steps with every kind of last step, unaligned rows."""
    _general_case(131, 139, K, ab=ab, la=la, lb=lb, pad=(1, 3, 1), ints=True)


@pytest.mark.parametrize("la,lb", LAYOUTS)
@pytest.mark.parametrize("ab", ["f16", "f32"])
@pytest.mark.parametrize("M,N", [(1, 1), (3, 7), (7, 3), (8, 9), (9, 8), (127, 135), (136, 257), (255, 129)])
def test_row_and_column_edges(la, lb, ab, M, N):
    """Dimensions shorter than a chunk, straddling the end of a chunk, a wave tile and a tile."""
    _general_case(M, N, 165, ab=ab, la=la, lb=lb, ints=True)
    _general_case(M, N, 100, ab=ab, la=la, lb=lb, batch=3, pad=(5, 1, 0), offset=1, ints=True)


@pytest.mark.parametrize("la,lb", LAYOUTS)
def test_slices_of_an_unaligned_sum(la, lb):
    """Slices of whole K steps, the last one with the partial step."""
    for K, split in ((1000, 3), (645, 5), (130, 2)):
        desc = P.make_desc(c_dtype="f32", layout_a=la, layout_b=lb, split_k=split)
        lda, ldb = (K if la == "row" else 75), (83 if lb == "row" else K)
        s, plan = P.prism_gemm_plan(desc, 75, 83, K, None, lda, 0, None, ldb, 0, None, 83, 0, 1)
        assert s == 0 and plan.kernel == 1 and plan.split_k > 1
        _general_case(75, 83, K, la=la, lb=lb, split_k=split, ints=True)
