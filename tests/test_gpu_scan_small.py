"""The scans without a chain of status words: sizes around their tiles and around the lines where
one way takes over from the other, in place and not, unaligned pointers, a workspace of exactly the
size asked for with guard words behind it, the same result as the chain gives."""
import numpy as np
import pytest
import torch

import paper_2511_11939_amd as P
from oracle import inclusive_scan_u32_ref
from workloads import scan_input_u32

pytestmark = pytest.mark.gpu
ALONE, PASS_TILE, TWO_PASS = 32768, 8192, 1 << 24


@pytest.mark.parametrize("n", [1, 5, 4095, 4097, ALONE - 1, ALONE, ALONE + 1, 5 * PASS_TILE - 1, 5 * PASS_TILE, 5 * PASS_TILE + 3,
                               1025 * PASS_TILE + 7, TWO_PASS, TWO_PASS + 1])
@pytest.mark.parametrize("in_place,offset", [(True, 0), (False, 1)])
def test_sizes_around_tiles_and_lines(n, in_place, offset):
    x = scan_input_u32(n, n)
    data = torch.zeros(n + offset, dtype=torch.int32, device="cuda")
    data[offset:] = torch.from_numpy(x.view(np.int32)).cuda()
    out = data if in_place else torch.full((n + offset,), -1, dtype=torch.int32, device="cuda")
    s, nbytes = P.prism_scan_workspace_size(n)
    assert s == 0
    ws = torch.full((nbytes + 64,), 0x5A, dtype=torch.uint8, device="cuda")
    stream = torch.cuda.current_stream().cuda_stream
    assert P.prism_scan_u32(data.data_ptr() + 4 * offset, out.data_ptr() + 4 * offset, n, ws, nbytes, stream) == 0
    assert P.prism_scan_check(ws, stream) == 0
    assert bool((ws[nbytes:] == 0x5A).all())
    got = out.cpu().numpy().view(np.uint32)
    assert (got[offset:] == inclusive_scan_u32_ref(x)).all()
    assert offset == 0 or got[0] == (0xFFFFFFFF if not in_place else 0)
