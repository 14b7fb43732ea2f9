"""Host-only: problems that one launch of the kernel for few rows could not take stay on tiles."""
import paper_2511_11939_amd as P


def _plan(M, N, K, batch=1):
    s, plan = P.prism_gemm_plan(P.make_desc(), M, N, K, None, K, M * K, None, K, K * N, None, N, M * N, batch)
    assert s == P.Status.OK
    return plan


def test_very_wide_and_very_many_problems_are_still_accepted():
    assert _plan(1, 1 << 25, 64).kernel == 4
    assert _plan(1, (1 << 31) - 128, 64).kernel == 2
    assert _plan(16, 16, 64, batch=1 << 21).kernel == 4
    assert _plan(16, 16, 64, batch=1 << 23).kernel != 4
