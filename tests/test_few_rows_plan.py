"""Host-only: which products of few rows take the kernel without tiles.  Problems that one launch of it could
not take stay on tiles, and so do those that tiles and a split are predicted to be faster at."""
import paper_2511_11939_amd as P


def _plan(M, N, K, batch=1, **kw):
    s, plan = P.prism_gemm_plan(P.make_desc(**kw), M, N, K, None, K, M * K, None, K, K * N, None, N, M * N, batch)
    assert s == P.Status.OK
    return plan


def test_very_wide_and_very_many_problems_are_still_accepted():
    assert _plan(1, 1 << 25, 64).kernel == 4
    assert _plan(1, (1 << 31) - 128, 64).kernel == 2
    assert _plan(16, 16, 64, batch=1 << 21).kernel == 4
    assert _plan(16, 16, 64, batch=1 << 23).kernel != 4


def test_a_long_way_for_few_workgroups_is_split_whatever_the_alignment():
    for K in (16384, 16383, 59410):
        plan = _plan(54, 52, K)
        assert plan.kernel in (1, 2) and plan.split_k >= 8, K
    assert _plan(56, 584, 59, batch=125).kernel == 1          # many rounds of short loops
    assert _plan(54, 52, 2000).kernel == 4 and _plan(16, 4096, 4096).kernel == 4


def test_without_a_split_there_is_no_reason_for_tiles():
    assert _plan(64, 512, 16384).split_k > 1
    for M, N, K in ((64, 512, 16384), (16, 512, 65536), (54, 52, 59410)):
        assert _plan(M, N, K, split_k=1).kernel == 4
