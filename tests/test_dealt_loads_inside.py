"""Which narrow operands the kernel that deals K steps to waves may take: its 16-byte loads of k-rows are
not bounded one by one, so the host must refuse every shape where one would leave the operand.  The
loads of a call are worked out here from its plan alone (no GPU)."""
import pytest

import paper_2511_11939_amd as P


def _k_row_loads(extent, ld, K, step, epc, tile, slice_k, other_runs_over):
    """(first, end) elements that the loads of a [K][extent] operand touch, first and last ones of every step."""
    for k_begin in range(0, K, slice_k):
        k_end = min(K, k_begin + slice_k)
        steps = (k_end - k_begin) // step
        over = k_end == K and steps * step == k_end - k_begin and (extent % epc != 0 or other_runs_over)
        whole = steps - (1 if over else 0)
        for x0 in range(0, extent, tile):
            rows = min(extent - x0, tile)
            for k in (k_begin, k_begin + whole * step - 1) if whole else ():   # whole steps: chunks as they come
                yield k * ld + x0, k * ld + x0 + (rows - 1) // epc * epc + epc
            rest = k_begin + whole * step
            for k in (rest, k_end - 1) if rest < k_end else ():                # the rest: chunks that end with the row
                yield k * ld + x0 + min(0, rows - epc), k * ld + x0 + rows


@pytest.mark.parametrize("ab,epc,step", [("f16", 8, 64), ("f32", 4, 32)])
@pytest.mark.parametrize("la,lb", [("row", "row"), ("col", "col"), ("col", "row")])
def test_loads_stay_inside(ab, epc, step, la, lb):
    taken = narrow = 0
    for M in (1, 3, 7, 33, 70, 129) if la == "col" else (70,):
        for N in (1, 2, 5, 7, 9, 33, 65, 131) if lb == "row" else (70,):
            for K in (1, epc, step - 1, step, step + 1, step + 2, step + 5, 2 * step, 3 * step - 1, 1003, 4096, 9001):
                for pad in (0, 1, 5):
                    lda, ldb = (M + pad if la == "col" else K), (N + pad if lb == "row" else K)
                    desc = P.make_desc(ab_dtype=ab, c_dtype="f32", layout_a=la, layout_b=lb)
                    s, plan = P.prism_gemm_plan(desc, M, N, K, None, lda, lda * K, None, ldb, ldb * K, None, N, M * N, 1)
                    assert s == 0
                    if plan.kernel not in (1, 2) or plan.tile_n >= 128:
                        continue
                    taken += 1
                    assert not plan.swapped
                    slice_k = -(-(-(-K // step)) // plan.split_k) * step
                    # (rows one element apart are contiguous along K)
                    a_rows, b_rows = la == "col" and lda > 1, lb == "row" and ldb > 1
                    for k_rows, extent, ld, other in ((a_rows, M, lda, b_rows and N % epc != 0), (b_rows, N, ldb, a_rows and M % epc != 0)):
                        if not k_rows:
                            assert K >= epc
                            continue
                        narrow += extent < epc
                        for first, end in _k_row_loads(extent, ld, K, step, epc, plan.tile_n, slice_k, other):
                            assert 0 <= first and end <= (K - 1) * ld + extent, (M, N, K, pad, first, end)
    assert taken > 20 and narrow > 0
