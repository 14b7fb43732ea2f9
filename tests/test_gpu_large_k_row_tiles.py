"""256x256 tiles with operands that are not contiguous along K (row-major B, column-major A, both):
K loops of one to five steps, sizes that end inside a tile, a wave tile and a block, batches and
K slices.  Exact on integers, and the race-check build gives the same bits for a row-major B (for the
other layouts in test_gpu_race_check_layouts)."""
import pytest

import paper_2511_11939_amd as P
from test_gpu_parity import _general_case
from test_gpu_paranoid_barriers import paranoid, test_paranoid_build_gives_the_same_bits as _same_bits  # noqa: F401

pytestmark = pytest.mark.gpu
LAYOUTS = [("row", "row"), ("col", "col"), ("col", "row")]


def _plan(la, lb, M, N, K, **kw):
    desc = P.make_desc(c_dtype="f32", layout_a=la, layout_b=lb, **kw)
    s, plan = P.prism_gemm_plan(desc, M, N, K, None, K if la == "row" else M, 0, None, N if lb == "row" else K, 0, None, N, 0, 1)
    assert s == 0
    return plan


@pytest.mark.parametrize("la,lb", LAYOUTS)
@pytest.mark.parametrize("ksteps", [1, 2, 3, 4, 5])
def test_k_loops_and_edges(la, lb, ksteps, set_hook):
    set_hook("PRISM_GEMM_CONFIG", "0")
    for M, N in ((256, 256), (264, 520), (104, 392)):
        plan = _plan(la, lb, M, N, 64 * ksteps)
        assert plan.kernel == 2 and plan.tile_m == 256 and plan.tile_n == 256
        _general_case(M, N, 64 * ksteps, la=la, lb=lb, ints=True)
    _general_case(264, 520, 64 * ksteps, la=la, lb=lb, ab="f16", cd="bf16", bias=True, alpha=-1.25, beta=0.5, batch=2, pad=(8, 16, 4))


@pytest.mark.parametrize("la,lb", LAYOUTS)
def test_slices_and_column_major_results(la, lb, set_hook):
    set_hook("PRISM_GEMM_CONFIG", "0")
    _general_case(264, 272, 832, la=la, lb=lb, split_k=3, ints=True)
    _general_case(264, 272, 320, la=la, lb=lb, lc="col", cd="f16", bias=True)


@pytest.mark.parametrize("la,lb", LAYOUTS)
def test_the_rule_takes_large_tiles_where_they_fill_the_chip(la, lb):
    assert _plan(la, lb, 4096, 4096, 256).tile_m == 256
    assert _plan(la, lb, 1024, 1280, 256).tile_m == 128
    _general_case(2944, 3080, 192, la=la, lb=lb, ints=True)      # 12 x 13 tiles, both directions with a remainder


def test_race_check_build(paranoid, set_hook):
    _same_bits(paranoid, set_hook, 768, 512, 448, 2, "row", "bf16", {"PRISM_GEMM_CONFIG": "0"})
