"""The scan with a chain of status words, which takes over beyond 2^24 elements: sizes around its tile of
16384, every combination of aligned and unaligned pointers, in place and not, a workspace that an
earlier scan of another size or kind has left full of stale words, replays from a graph, and the entry
point whose status words are the library's own."""
import numpy as np
import pytest
import torch

import paper_2511_11939_amd as P
from oracle import inclusive_scan_u32_ref
from workloads import scan_input_u32

pytestmark = pytest.mark.gpu
TILE, LINE = 16384, 1 << 24


def _workspace(n):
    s, nbytes = P.prism_scan_workspace_size(n)
    assert s == 0
    return torch.full((nbytes,), 0x5A, dtype=torch.uint8, device="cuda")


def _device(x, offset):
    data = torch.zeros(x.size + offset, dtype=torch.int32, device="cuda")
    data[offset:] = torch.from_numpy(x.view(np.int32)).cuda()
    return data


def _check(out, offset, x, rest):
    got = out.cpu().numpy().view(np.uint32)
    assert (got[offset:offset + x.size] == inclusive_scan_u32_ref(x)).all()
    assert (got[:offset] == rest).all() and (got[offset + x.size:] == rest).all()


@pytest.mark.parametrize("n", [LINE + 1, LINE + TILE - 1, LINE + TILE, LINE + TILE + 1, LINE + 70 * TILE + 777])
@pytest.mark.parametrize("offset_in,offset_out,in_place", [(0, 0, True), (1, 1, True), (0, 1, False), (3, 0, False), (2, 3, False)])
def test_sizes_and_pointers(n, offset_in, offset_out, in_place):
    x = scan_input_u32(n & 0xFFFF, n)
    data = _device(x, offset_in)
    out = data if in_place else torch.full((n + offset_out + 5,), -1, dtype=torch.int32, device="cuda")
    ws = _workspace(n)
    P.scan_u32(data.data_ptr() + 4 * offset_in, out.data_ptr() + 4 * offset_out, n, ws)
    assert P.prism_scan_check(ws, torch.cuda.current_stream().cuda_stream) == 0
    _check(out, offset_out, x, 0 if in_place else 0xFFFFFFFF)


def test_a_workspace_full_of_stale_words():
    """Prefixes of another array, the sums of the scan without a chain, then the chain again."""
    n = LINE + 33 * TILE + 5
    ws = _workspace(n)
    for seed, size in ((1, n), (2, n), (3, 40 * TILE + 9), (4, n - TILE), (5, 1000), (6, n)):
        x = scan_input_u32(seed, size)
        data, out = _device(x, 0), torch.full((size,), -1, dtype=torch.int32, device="cuda")
        P.scan_u32(data, out, size, ws)
        assert P.prism_scan_check(ws, torch.cuda.current_stream().cuda_stream) == 0
        _check(out, 0, x, 0)


@pytest.mark.parametrize("static", [False, True])
def test_replays_from_a_graph(static):
    n = LINE + 9 * TILE + 77
    x = scan_input_u32(31, n)
    data, out, ws = _device(x, 0), torch.empty(n, dtype=torch.int32, device="cuda"), _workspace(n)
    flag = torch.full((1,), 7, dtype=torch.int32, device="cuda")

    def enqueue(stream):
        if static:
            assert P.prism_scan_u32_static(data, out, n, flag, stream.cuda_stream) == 0
        else:
            P.scan_u32(data, out, n, ws, stream=stream)

    enqueue(torch.cuda.current_stream())      # eager first (the library's own array is looked up once per device)
    torch.cuda.synchronize()
    _check(out, 0, x, 0)
    side, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side), torch.cuda.graph(graph, stream=side):
        enqueue(side)
    for _ in range(4):
        out.fill_(-1)                          # eager work between the replays
        ws.fill_(0x5A)
        flag.fill_(7)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        _check(out, 0, x, 0)
        if static:
            assert int(flag.item()) == 0
        else:
            assert P.prism_scan_check(ws, torch.cuda.current_stream().cuda_stream) == 0


def test_the_library_s_own_status_words_twice_in_a_row():
    flag = torch.full((1,), 7, dtype=torch.int32, device="cuda")
    stream = torch.cuda.current_stream().cuda_stream
    arrays = [scan_input_u32(40 + i, n) for i, n in enumerate((LINE + 50 * TILE + 1, LINE + TILE // 2, 3 * TILE, LINE + 2))]
    data = [_device(x, i & 1) for i, x in enumerate(arrays)]
    outs = [torch.full((x.size,), -1, dtype=torch.int32, device="cuda") for x in arrays]
    for i, x in enumerate(arrays):            # nothing in between
        assert P.prism_scan_u32_static(data[i].data_ptr() + 4 * (i & 1), outs[i], x.size, flag, stream) == 0
    torch.cuda.synchronize()
    assert int(flag.item()) == 0
    for x, out in zip(arrays, outs):
        _check(out, 0, x, 0)
