"""The epilogue's three forms (whole tile plain, whole tile with beta or a bias per row, edge) on
every kernel that has one, with rows of C at every alignment: odd leading dimensions, offset
pointers, tiles that end inside a block, inside a run of four columns and inside a run of eight."""
import pytest

from test_gpu_parity import _general_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cd", ["bf16", "f16", "f32"])
@pytest.mark.parametrize("M,N", [(128, 128), (129, 130), (257, 133), (130, 135), (65, 67), (192, 196)])
@pytest.mark.parametrize("beta,bias,lc", [(0.0, False, "row"), (0.0, True, "row"), (0.0, True, "col"), (-0.75, True, "row"), (0.5, False, "col")])
def test_pipeline_and_staged_store_any_shape(cd, M, N, beta, bias, lc):
    for lb, K, pads in (("col", 128, (0, 0, 0)), ("row", 100, (1, 1, 3)), ("col", 70, (0, 0, 1))):
        _general_case(M, N, K, cd=cd, lb=lb, lc=lc, beta=beta, bias=bias, pad=pads, alpha=1.5, seed=M + N)


@pytest.mark.parametrize("cfg,persistent", [("0", "0"), ("0", "1"), ("1", "0")])
@pytest.mark.parametrize("cd", ["bf16", "f32"])
def test_large_tiles_and_the_persistent_kernel(cfg, persistent, cd, set_hook):
    set_hook("PRISM_GEMM_CONFIG", cfg)
    set_hook("PRISM_PERSISTENT", persistent)
    for M, N, pad, kw in ((512, 256, 0, dict(beta=0.5)), (300, 261, 3, dict(bias=True)), (261, 300, 1, dict(bias=True, lc="col", beta=-1.0)),
                          (256, 512, 1, dict(bias=True)), (255, 253, 0, dict())):
        _general_case(M, N, 128, cd=cd, pad=(0, 0, pad), alpha=0.5, batch=2, **kw)


@pytest.mark.parametrize("N", [63, 64, 65, 66, 131])
def test_partial_sums_of_any_width(N):
    _general_case(70, N, 640, split_k=4, ints=True)
    _general_case(70, N, 640, split_k=4, cd="bf16", bias=True, beta=0.5, lc="col", pad=(0, 0, 1))
    _general_case(70, N, 640, split_k=5, cd="f16", bias=True, beta=0.5, pad=(0, 0, 1))
