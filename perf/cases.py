"""The work that users of this library have it do, as cases that can be timed and compared.

A case is a dict of plain values: a matrix product through `gemm` (sizes, types, layouts, scalars)
or a prefix sum through `scan_u32`.  `listed()` names the cases that are always measured, `draw`
gives more of the same ranges, `prepare` makes what a user's program holds before the call,
`run` is one call through the public entry points, `exact` the same in 64 bits with plain torch.
"""
import math

import torch

import paper_2511_11939_amd as P

_TORCH_TYPE = {"bf16": torch.bfloat16, "f16": torch.float16, "f32": torch.float32}
_BYTES = {"bf16": 2, "f16": 2, "f32": 4}


def _gemm(M, N, K, *, batch=1, ab="bf16", c="bf16", la="row", lb="col", lc="row", alpha=1.0, beta=0.0, bias=False,
          values="normal", name=None):
    case = {"op": "gemm", "M": M, "N": N, "K": K, "batch": batch, "ab": ab, "c": c, "la": la, "lb": lb, "lc": lc,
            "alpha": alpha, "beta": beta, "bias": bias, "values": values}
    return case if name is None else {"name": name, **case}


def _scan(n, *, in_place=False, name=None):
    case = {"op": "scan", "n": n, "in_place": in_place}
    return case if name is None else {"name": name, **case}


def listed():
    return [
        # the smallest call: one product of 256 x 256 matrices, everything row-major, fp32 result;
        # a program that makes many of these waits for launches
        _gemm(256, 256, 256, c="f32", lb="row", values="uniform", name="small_256_rowrow"),
        # decoding: the weights of a 4096 x 4096 projection against sixteen tokens, bias fused
        _gemm(16, 4096, 4096, bias=True, values="weights", name="decode_16x4096x4096"),
        # odd sizes, packed rows: nothing is aligned and no dimension is a multiple of a tile
        _gemm(1999, 2001, 1003, name="ragged_1999x2001x1003"),
        # the library's headline: a square bf16 product
        _gemm(4096, 4096, 4096, name="square_4096"),
        # prefill: 16384 tokens through a 4096 x 4096 projection with its bias
        _gemm(16384, 4096, 4096, bias=True, values="weights", name="projection_16384x4096"),
        # the projection's backward pass: the input's gradient (the weights are row-major here) ...
        _gemm(8192, 4096, 4096, lb="row", values="weights", name="input_gradient_8192x4096"),
        # ... and the weights' gradient, summed over tokens and accumulated in fp32
        _gemm(4096, 4096, 8192, c="f32", la="col", lb="row", beta=1.0, name="weight_gradient_4096x8192"),
        # few results, a very long sum: fp16, split over K and reduced on the device
        _gemm(1024, 1024, 32768, ab="f16", c="f32", values="uniform", name="long_sum_1024x32768"),
        # many small independent products in one call
        _gemm(512, 512, 512, batch=256, name="batched_256x512"),
        # the fp32 product of the paper's sgemm study, all matrices row-major, both scalars in use
        _gemm(4096, 4096, 4096, ab="f32", c="f32", lb="row", alpha=1.5, beta=0.5, values="uniform", name="sgemm_4096"),
        # prefix sums: a small array of odd length, summed in place as the paper's kernel does ...
        _scan(1000003, in_place=True, name="scan_1000003"),
        # ... and an array far beyond every cache
        _scan(1 << 28, name="scan_2p28"),
    ]


def _log_int(rng, lo, hi):
    """A whole number of [lo, hi], spread over its logarithm."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _size(rng, lo, hi):
    """A size of [lo, hi]: half of them whole multiples of 64 (or powers of two below that), the others as they come."""
    v = _log_int(rng, lo, hi)
    if rng.random() < 0.5:
        return v
    return max(64, (v + 32) // 64 * 64) if v >= 64 else 1 << (v.bit_length() - 1)


def draw(rng):
    """One more case of the ranges that the listed ones stand for."""
    kind = rng.choice(["ordinary", "ordinary", "decode", "ragged", "prefill", "backward", "long", "batched", "fp32", "scan", "scan"])
    half = rng.choice(["bf16", "bf16", "f16"])
    if kind == "scan":
        return _scan(_log_int(rng, 1000, 1 << 28), in_place=rng.random() < 0.5)
    while True:
        if kind == "ordinary":      # products of a few hundred to a few thousand rows and columns
            case = _gemm(_size(rng, 128, 4096), _size(rng, 128, 4096), _size(rng, 128, 4096), ab=half, c=rng.choice([half, "f32"]),
                         lb=rng.choice(["col", "row"]), bias=rng.random() < 0.3)
        elif kind == "decode":      # 1 to 128 tokens against a weight matrix
            case = _gemm(_log_int(rng, 1, 128), _size(rng, 512, 16384), 64 * _log_int(rng, 8, 256), ab=half, c=half,
                         bias=rng.random() < 0.5, values="weights")
        elif kind == "ragged":      # any sizes, any layouts
            case = _gemm(_log_int(rng, 17, 3000), _log_int(rng, 17, 3000), _log_int(rng, 17, 3000), ab=half, c=rng.choice([half, "f32"]),
                         la=rng.choice(["row", "col"]), lb=rng.choice(["row", "col"]), lc=rng.choice(["row", "row", "col"]),
                         alpha=rng.choice([1.0, 0.5]), beta=rng.choice([0.0, 0.0, 1.0]), bias=rng.random() < 0.3)
        elif kind == "prefill":     # many tokens through a projection
            case = _gemm(_log_int(rng, 512, 16384), 64 * _log_int(rng, 8, 160), 64 * _log_int(rng, 8, 160), ab=half, c=half,
                         bias=rng.random() < 0.5, values="weights")
        elif kind == "backward":    # its gradients
            tokens, n, k = 64 * _log_int(rng, 8, 256), 64 * _log_int(rng, 8, 128), 64 * _log_int(rng, 8, 128)
            case = (_gemm(tokens, n, k, ab=half, c=half, lb="row", values="weights") if rng.random() < 0.5 else
                    _gemm(n, k, tokens, ab=half, c="f32", la="col", lb="row", beta=rng.choice([0.0, 1.0])))
        elif kind == "long":        # few results, long sums
            case = _gemm(64 * _log_int(rng, 1, 16), 64 * _log_int(rng, 1, 16), 64 * _log_int(rng, 64, 1024), ab=half, c="f32",
                         values="uniform")
        elif kind == "batched":     # many small independent products
            case = _gemm(_size(rng, 32, 1024), _size(rng, 32, 1024), _size(rng, 32, 1024), batch=_log_int(rng, 2, 256), ab=half,
                         c=rng.choice([half, "f32"]))
        else:                       # fp32 operands
            case = _gemm(_size(rng, 32, 4096), _size(rng, 32, 4096), _size(rng, 32, 4096), ab="f32", c="f32",
                         la=rng.choice(["row", "row", "col"]), lb=rng.choice(["row", "col"]), alpha=rng.choice([1.0, 1.5]),
                         beta=rng.choice([0.0, 0.5]), values="uniform")
        flops = 2.0 * case["M"] * case["N"] * case["K"] * case["batch"]
        aligned = case["M"] % 64 == 0 and case["N"] % 64 == 0 and case["K"] % 64 == 0
        limit = 1.0e11 if case["ab"] == "f32" and aligned else 5.4e11 if kind in ("prefill", "backward") else 1.3e11 if aligned else 4.0e10
        if flops <= limit:
            return case


def _span(rows, cols, layout, batch):
    return (batch, rows, cols) if layout == "row" else (batch, cols, rows)


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    if case["op"] == "scan":
        n = case["n"]
        x = torch.randint(-2 ** 31, 2 ** 31, (n,), dtype=torch.int32, device="cuda", generator=gen)
        status, nbytes = P.prism_scan_workspace_size(n)
        assert status == P.Status.OK
        return {"case": case, "x": x, "out": x if case["in_place"] else torch.empty_like(x),
                "workspace": torch.empty(nbytes, dtype=torch.uint8, device="cuda")}

    M, N, K, batch = (case[k] for k in ("M", "N", "K", "batch"))

    def values(shape, scale):
        if case["values"] == "uniform":
            return torch.empty(shape, device="cuda").uniform_(-1.0, 1.0, generator=gen)
        return torch.empty(shape, device="cuda").normal_(0.0, scale, generator=gen)

    kind = _TORCH_TYPE[case["ab"]]
    A = values(_span(M, K, case["la"], batch), 1.0).to(kind)
    B = values(_span(K, N, case["lb"], batch), 0.02 if case["values"] == "weights" else 1.0).to(kind)
    C = torch.empty(_span(M, N, case["lc"], batch), dtype=_TORCH_TYPE[case["c"]], device="cuda")
    if case["beta"] != 0.0:
        C.normal_(0.0, 1.0, generator=gen)
    bias = torch.empty(N, device="cuda").normal_(0.0, 1.0, generator=gen) if case["bias"] else None
    desc = P.make_desc(ab_dtype=case["ab"], c_dtype=case["c"], layout_a=case["la"], layout_b=case["lb"], layout_c=case["lc"],
                       alpha=case["alpha"], beta=case["beta"], bias=bias)
    status, nbytes = P.prism_gemm_workspace_size(desc, M, N, K, batch)
    assert status == P.Status.OK
    workspace = torch.empty(nbytes, dtype=torch.uint8, device="cuda") if nbytes else None
    if workspace is not None:
        desc.workspace, desc.workspace_bytes = workspace.data_ptr(), nbytes
    return {"case": case, "A": A, "B": B, "C": C, "bias": bias, "desc": desc, "workspace": workspace}


def run(state):
    case = state["case"]
    if case["op"] == "scan":
        P.scan_u32(state["x"], state["out"], case["n"], state["workspace"])
        return state["out"]
    P.gemm(state["A"], state["B"], state["C"], M=case["M"], N=case["N"], K=case["K"], desc=state["desc"], batch=case["batch"])
    return state["C"]


def work(case):
    if case["op"] == "scan":
        return {"bytes": 8.0 * case["n"], "flops": 0.0}
    M, N, K, batch = (case[k] for k in ("M", "N", "K", "batch"))
    c_bytes = M * N * _BYTES[case["c"]] * (2 if case["beta"] != 0.0 else 1)
    return {"bytes": float(batch * ((M * K + K * N) * _BYTES[case["ab"]] + c_bytes) + (4 * N if case["bias"] else 0)),
            "flops": 2.0 * M * N * K * batch}


def tolerance(case):
    if case["op"] == "scan":
        return "exact"  # sums of whole numbers modulo 2^32
    # 16-bit results: one rounding of the fp32 value (measured against 64 bits: 1.7e-3 for bf16, 2.1e-4 for fp16)
    if case["c"] == "bf16":
        return {"rel": 6.5e-3}
    if case["c"] == "f16":
        return {"rel": 8.0e-4}
    # fp32 results: the order of the sums; the error of a sum in order grows with its length
    # (measured against 64 bits: 1.1e-6 for fp32 operands at K = 4096, 8e-8 at K = 256)
    return {"rel": 3.0e-7 + 7.0e-8 * math.sqrt(case["K"])}


def exact(case, seed):
    state = prepare(case, seed)
    if case["op"] == "scan":
        total = torch.cumsum(state["x"].to(torch.int64) & 0xFFFFFFFF, 0) & 0xFFFFFFFF
        return torch.where(total >= 2 ** 31, total - 2 ** 32, total).to(torch.int32)
    A, B, C = state["A"].double(), state["B"].double(), state["C"].double()
    A = A if case["la"] == "row" else A.transpose(1, 2).contiguous()
    B = B if case["lb"] == "row" else B.transpose(1, 2).contiguous()
    out = torch.stack([case["alpha"] * (A[i] @ B[i]) for i in range(case["batch"])])
    if case["bias"]:
        out += state["bias"].double()
    out = out if case["lc"] == "row" else out.transpose(1, 2).contiguous()
    return out + case["beta"] * C if case["beta"] != 0.0 else out
