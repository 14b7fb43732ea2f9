"""Host-only: which tile operands that are not contiguous along K get.  Large tiles must not leave the chip
idle where small ones would fill it: sums over very many tokens, tiles that are mostly beyond
the matrix, loops of a few K steps."""
import pytest

import paper_2511_11939_amd as P

LAYOUTS = [("row", "row"), ("col", "col"), ("col", "row")]


def _plan(la, lb, M, N, K, batch=1, **kw):
    desc = P.make_desc(c_dtype="f32", layout_a=la, layout_b=lb, **kw)
    s, plan = P.prism_gemm_plan(desc, M, N, K, None, K if la == "row" else M, M * K, None, N if lb == "row" else K, K * N, None, N, M * N, batch)
    assert s == P.Status.OK and plan.kernel == 2
    return plan


@pytest.mark.parametrize("la,lb", LAYOUTS)
@pytest.mark.parametrize("M,N,K,workgroups", [(256, 256, 32768, 128), (256, 256, 65536, 128), (512, 512, 32768, 512), (192, 640, 40960, 300)])
def test_few_tiles_and_a_very_long_sum_fill_the_chip(la, lb, M, N, K, workgroups):
    plan = _plan(la, lb, M, N, K)
    assert plan.tile_m == 128 and plan.workgroups >= workgroups


@pytest.mark.parametrize("la,lb", LAYOUTS)
def test_large_tiles_that_hold_little_stay_small(la, lb):
    assert _plan(la, lb, 744, 64, 64, batch=58).tile_m == 128     # a quarter of every large tile
    assert _plan(la, lb, 1408, 896, 64, batch=8).tile_m == 128    # one K step
    assert _plan(la, lb, 256, 3264, 128, batch=30).tile_m == 128  # rounds of two steps
    assert _plan(la, lb, 768, 1984, 192, batch=10).tile_m == 128  # two rounds of three steps, nearly full


@pytest.mark.parametrize("la,lb", LAYOUTS)
def test_gradients_keep_large_tiles(la, lb):
    assert _plan(la, lb, 8192, 4096, 4096).tile_m == 256
    assert _plan(la, lb, 4096, 4096, 8192).tile_m == 256
    assert _plan(la, lb, 2048, 2048, 65536).tile_m == 256


@pytest.mark.parametrize("la,lb", LAYOUTS)
def test_more_small_tiles_than_a_launch_takes(la, lb):
    M = N = 128 * 6000
    assert _plan(la, lb, M, N, 64).tile_m == 256
