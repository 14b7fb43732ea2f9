"""Host-only: the native way of the usual call gives the status that the way through ctypes gives, for every form
of its arguments that it takes, and declines all others.  Problems that are empty or refused on the
host, so that nothing is launched."""
import ctypes
import itertools

import numpy as np
import pytest
import torch

import paper_2511_11939_amd as P
from paper_2511_11939_amd import _call, binding

A, B, C = (torch.zeros(1 << 16, dtype=torch.int16) for _ in range(3))


@pytest.fixture(autouse=True)
def _bound_without_a_gpu():
    lib = P.load_library()
    address = [ctypes.cast(f, ctypes.c_void_p).value for f in (lib.prism_gemm, lib.prism_gemm_batched, lib.prism_scan_u32)]
    _call.bind(*address, P.GemmDesc, lambda: 0, lambda device: 0)
    yield
    binding._call = None  # bound anew, to torch, by the next call


def _both(M, N, K, desc, *ld_batch_strides):
    lda, ldb, ldc, batch, *strides = ld_batch_strides
    native = _call.gemm(A, B, C, M, N, K, desc, lda, ldb, ldc, batch, *strides)
    try:  # a stream that is given takes the way through ctypes
        P.gemm(A, B, C, M=M, N=N, K=K, desc=desc, lda=lda, ldb=ldb, ldc=ldc, batch=batch, strideA=strides[0], strideB=strides[1],
               strideC=strides[2], stream=0)
        return native, 0
    except P.PrismError as e:
        return native, int(e.status)


def test_the_same_status_for_every_form():
    seen = set()
    for layouts in itertools.product(("row", "col"), repeat=3):
        desc = P.make_desc(layout_a=layouts[0], layout_b=layouts[1], layout_c=layouts[2], c_dtype="f32")
        for M, N, K in ((0, 5, 7), (5, 0, 0), (0, 0, 0), (8, 16, 32)):
            for lds in ((None, None, None), (0, None, -3), (3, 4, 5), (64, 64, 2)):
                for batch, strides in ((1, (None, None, None)), (0, (None, None, None)), (3, (None, None, 1)), (1, (0, None, 0)), (-1, (5, 6, 7))):
                    if M and N and not (batch == -1 or lds == (3, 4, 5) or lds == (64, 64, 2) or (batch == 3 and strides[2] == 1)):
                        continue                                # (would be launched)
                    if M and N and lds == (64, 64, 2) and layouts[2] == "row" and 2 >= N or batch == 0 and lds[0] is None and M and N:
                        continue
                    native, other = _both(M, N, K, desc, *lds, batch, *strides)
                    assert native == other, (layouts, M, N, K, lds, batch, strides)
                    seen.add(native)
    desc = P.make_desc(ab_dtype="f32", c_dtype="bf16")
    assert _both(4, 4, 4, desc, None, None, None, 1, None, None, None) == (2, 2)
    assert {0, 1} <= seen


def test_everything_else_is_declined():
    desc = P.make_desc()
    usual = [A, B, C, 0, 4, 4, desc, None, None, None, 1, None, None, None]
    assert _call.gemm(*usual) == 0
    for at, value in ((0, A.data_ptr()), (1, None), (2, "C"), (3, True), (3, np.int64(0)), (4, 1.0), (4, -1), (5, 1 << 40), (5, 1 << 80), (6, None),
                      (6, object()), (7, "4"), (8, 1 << 70), (10, np.int32(1)), (10, None), (11, 2.5)):
        assert _call.gemm(*usual[:at], value, *usual[at + 1:]) is None, (at, value)
    assert _call.gemm(*usual[:-1]) is None
    ws = torch.zeros(72, dtype=torch.uint8)
    assert _call.scan(A, A, 0, ws) == 0 and _call.scan(A, B, -1, ws) == 1 and _call.scan(A, B, 100, ws[:71]) == 3
    for args in ((A.data_ptr(), B, 0, ws), (A, B, np.int64(0), ws), (A, B, 0, None), (A, B, 0, ws.data_ptr()), (A, B, 1 << 65, ws), (A, B, 0)):
        assert _call.scan(*args) is None
