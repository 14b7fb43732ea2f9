"""Scans by one workgroup: sizes around the line between two and eight chunks per lane."""
import pytest
import torch

import paper_2511_11939_amd as P
from oracle import inclusive_scan_u32_ref
from workloads import scan_input_u32

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [63, 1024, 4096, 8189, 8191, 8192, 8193, 8196, 16384])
def test_sizes_around_the_line(n):
    x = scan_input_u32(n, n)
    data = torch.from_numpy(x.view("int32")).cuda()
    out = torch.full((n + 4,), -1, dtype=torch.int32, device="cuda")
    s, nbytes = P.prism_scan_workspace_size(n)
    ws = torch.full((nbytes,), 0x5A, dtype=torch.uint8, device="cuda")
    P.scan_u32(data, out, n, ws)
    assert P.prism_scan_check(ws, torch.cuda.current_stream().cuda_stream) == 0
    got = out.cpu().numpy().view("uint32")
    assert (got[:n] == inclusive_scan_u32_ref(x)).all() and (got[n:] == 0xFFFFFFFF).all()
