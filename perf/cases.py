"""The work that the library's speed is measured on.

Every case is one pass through the package's public entry points, as a program
that uses the library calls them: ``gemm`` on the five arithmetic paths,
``gemm_i8``, ``gemm_batched``, the differentiable ``matmul`` with its backward,
SYR2K, and the FP8 product on weights packed once.  ``listed()`` gives the
fixed cases, ``draw()`` further ones of the same ranges; a drawn size is odd or
ragged about half of the time, since a program's own matrices are seldom
multiples of a tile.
"""
from __future__ import annotations

import math

import torch

from paper_2305_18236_amd import _native, gemm, gemm_batched, gemm_i8
from paper_2305_18236_amd.autograd import matmul

# Sizes of one dimension that the families below cover (drawn evenly over the
# logarithm): small products, general ones, and the few rows of a skinny one.
SMALL = (16, 384)
GENERAL = (384, 6144)
ROWS = (1, 256)
WIDE = (1024, 8192)


def listed():
    return [
        # The paper's small size: one call's latency, a handful of workgroups.
        {"name": "fp32_256", "kind": "gemm", "path": "fp32", "M": 256, "N": 256, "K": 256, "layout": "NN",
         "beta": 0.0},
        # An ordinary update C <- AB + C/2 of the FP32 sweep's smallest size.
        {"name": "fp32_1024", "kind": "gemm", "path": "fp32", "M": 1024, "N": 1024, "K": 1024, "layout": "NN",
         "beta": 0.5},
        # Sizes that no tile divides and odd row strides, A stored transposed
        # (the product of a weight gradient).
        {"name": "fp32_ragged", "kind": "gemm", "path": "fp32", "M": 1531, "N": 2047, "K": 1021, "layout": "TN",
         "beta": 0.0},
        # The headline benchmark, the largest product.
        {"name": "fp32_8192", "kind": "gemm", "path": "fp32", "M": 8192, "N": 8192, "K": 8192, "layout": "NN",
         "beta": 0.0},
        # A few rows times a large stored-transposed weight matrix: reading
        # the weights bounds it.
        {"name": "fp32_skinny", "kind": "gemm", "path": "fp32", "M": 32, "N": 8192, "K": 8192, "layout": "NT",
         "beta": 0.0},
        # The same with weights quantised and packed once, the rows on each call.
        {"name": "fp8_decode", "kind": "fp8_packed", "M": 64, "N": 8192, "K": 8192},
        # One layer of the chain benchmark: forward and hand-written backward.
        {"name": "train_bf16x3", "kind": "train", "path": "bf16x3", "M": 4096, "N": 8192, "K": 2048},
        # A 16-bit product of ragged size, B stored transposed (a linear layer).
        {"name": "bf16_ragged", "kind": "gemm", "path": "bf16", "M": 2500, "N": 3001, "K": 1777, "layout": "NT",
         "beta": 0.0},
        # FP8 end to end: both operands quantised in the call.
        {"name": "fp8_4096", "kind": "gemm", "path": "fp8", "M": 4096, "N": 4096, "K": 4096, "layout": "NN",
         "beta": 0.0},
        # Integers of ragged size and odd row strides.
        {"name": "i8_ragged", "kind": "gemm_i8", "M": 2000, "N": 2501, "K": 3001, "layout": "NN", "beta": 0},
        # The batched benchmark: 512 products of uneven size in one launch.
        {"name": "batched_512", "kind": "batched", "path": "fp32", "count": 512, "lo": 32, "hi": 2048, "step": 8,
         "sizes_seed": 3},
        # The symmetric update of one triangle at an ordinary size.
        {"name": "syr2k_2048", "kind": "syr2k", "uplo": "L", "trans": "N", "N": 2048, "K": 2048, "beta": 0.5},
    ]


def _size(rng, span):
    """A size of `span`, even over its logarithm: as it comes, or rounded to
    a multiple of 8 or 64 as a program's chosen sizes often are."""
    lo, hi = span
    x = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    step = rng.choice((1, 1, 8, 64))
    if x > 4 * step:
        x = (x + step // 2) // step * step
    return min(max(x, lo), hi)


def draw(rng):
    kind = rng.choice(("small", "fp32", "fp32", "16bit", "16bit", "fp8", "i8", "skinny", "decode", "train", "batched",
                       "syr2k"))
    layout = rng.choice(("NN", "NT", "TN", "TT"))
    beta = rng.choice((0.0, 0.0, 0.5))
    if kind == "small":
        return {"kind": "gemm", "path": "fp32", "M": _size(rng, SMALL), "N": _size(rng, SMALL),
                "K": _size(rng, SMALL), "layout": layout, "beta": beta}
    if kind in ("fp32", "16bit", "fp8"):
        path = rng.choice(("bf16x3", "bf16", "fp16")) if kind == "16bit" else kind
        return {"kind": "gemm", "path": path, "M": _size(rng, GENERAL), "N": _size(rng, GENERAL),
                "K": _size(rng, GENERAL), "layout": layout, "beta": beta}
    if kind == "i8":
        return {"kind": "gemm_i8", "M": _size(rng, GENERAL), "N": _size(rng, GENERAL), "K": _size(rng, GENERAL),
                "layout": layout, "beta": rng.choice((0, 0, 1))}
    if kind == "skinny":
        return {"kind": "gemm", "path": "fp32", "M": _size(rng, ROWS), "N": _size(rng, WIDE), "K": _size(rng, WIDE),
                "layout": rng.choice(("NN", "NT")), "beta": 0.0}
    if kind == "decode":
        return {"kind": "fp8_packed", "M": _size(rng, ROWS), "N": _size(rng, WIDE), "K": _size(rng, WIDE)}
    if kind == "train":
        return {"kind": "train", "path": rng.choice(("fp32", "bf16x3", "bf16")), "M": _size(rng, GENERAL),
                "N": _size(rng, GENERAL), "K": _size(rng, (384, 4096))}
    if kind == "batched":
        return {"kind": "batched", "path": rng.choice(("fp32", "bf16x3", "bf16")), "count": _size(rng, (16, 512)),
                "lo": 32, "hi": rng.choice((512, 1024, 2048)), "step": rng.choice((1, 8)),
                "sizes_seed": rng.randrange(1000)}
    return {"kind": "syr2k", "uplo": rng.choice("LU"), "trans": rng.choice("NT"), "N": _size(rng, (384, 4096)),
            "K": _size(rng, (384, 4096)), "beta": beta}


def _batch_sizes(case):
    """M, N, K of each problem: exp of a uniform draw over [ln lo, ln hi], in
    steps of `step`, at least lo."""
    gen = torch.Generator().manual_seed(case["sizes_seed"])
    u = torch.rand((case["count"], 3), generator=gen, dtype=torch.float64)
    s = torch.exp(math.log(case["lo"]) + u * (math.log(case["hi"]) - math.log(case["lo"])))
    s = (s / case["step"]).round().mul(case["step"]).clamp(case["lo"], case["hi"])
    return [tuple(int(v) for v in row) for row in s.tolist()]


def _uniform(gen, *shape):
    return torch.empty(shape, device="cuda").uniform_(-1.0, 1.0, generator=gen)


def _operand(gen, rows, cols, trans, make=_uniform):
    """op(X) of rows x cols: stored so, or transposed and read through a view."""
    return make(gen, cols, rows).t() if trans == "T" else make(gen, rows, cols)


def _int8(gen, *shape):
    return torch.randint(-128, 128, shape, device="cuda", dtype=torch.int8, generator=gen)


def _slabs(gen, case):
    """The batch's operands and results as views of three slabs, each matrix
    beginning at a multiple of 64 elements."""
    sizes = _batch_sizes(case)
    pad = lambda n: -(-n // 64) * 64  # noqa: E731
    a = _uniform(gen, sum(pad(m * k) for m, _, k in sizes))
    b = _uniform(gen, sum(pad(k * n) for _, n, k in sizes))
    c = torch.zeros(sum(pad(m * n) for m, n, _ in sizes), device="cuda")
    views, ia, ib, ic = [], 0, 0, 0
    for m, n, k in sizes:
        views.append((a[ia:ia + m * k].view(m, k), b[ib:ib + k * n].view(k, n), c[ic:ic + m * n].view(m, n)))
        ia, ib, ic = ia + pad(m * k), ib + pad(k * n), ic + pad(m * n)
    return views, c


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(int(seed))
    kind = case["kind"]
    s = dict(case)
    if kind == "gemm":
        s["A"] = _operand(gen, case["M"], case["K"], case["layout"][0])
        s["B"] = _operand(gen, case["K"], case["N"], case["layout"][1])
        s["C"] = _uniform(gen, case["M"], case["N"]) if case["beta"] else None
    elif kind == "gemm_i8":
        s["A"] = _operand(gen, case["M"], case["K"], case["layout"][0], _int8)
        s["B"] = _operand(gen, case["K"], case["N"], case["layout"][1], _int8)
        s["C"] = (torch.randint(-1000, 1000, (case["M"], case["N"]), device="cuda", dtype=torch.int32, generator=gen)
                  if case["beta"] else None)
    elif kind == "fp8_packed":
        M, N, K = case["M"], case["N"], case["K"]
        s["X"] = _uniform(gen, M, K)
        s["W"] = _uniform(gen, N, K)
        for name, rows in (("x", M), ("w", N)):
            q, sc = _native.mg_fp8_packed_size(rows, K)
            s["q" + name] = torch.empty(q, dtype=torch.uint8, device="cuda")
            s["s" + name] = torch.empty(sc, dtype=torch.uint8, device="cuda")
        _native.check(_native.mg_fp8_pack("N", N, K, s["W"].data_ptr(), K, s["qw"].data_ptr(), s["sw"].data_ptr(),
                                          torch.cuda.current_stream().cuda_stream), "mg_fp8_pack")
        s["Y"] = torch.empty((M, N), device="cuda")
    elif kind == "train":
        s["X"] = _uniform(gen, case["M"], case["K"]).requires_grad_(True)
        s["W"] = _uniform(gen, case["K"], case["N"]).requires_grad_(True)
        s["G"] = torch.empty((case["M"], case["N"]), device="cuda").normal_(generator=gen)
    elif kind == "batched":
        views, s["C"] = _slabs(gen, case)
        s["problems"] = [(a, b, c, 1.0, 0.0) for a, b, c in views]
    else:
        N, K = case["N"], case["K"]
        shape = (N, K) if case["trans"] == "N" else (K, N)
        s["A"], s["B"] = _uniform(gen, *shape), _uniform(gen, *shape)
        s["C"] = _uniform(gen, N, N)
        s["bytes"] = _native.mg_syr2k_workspace_size(0, N, K)
        s["workspace"] = torch.empty(max(s["bytes"], 1), dtype=torch.uint8, device="cuda")
    return s


def run(s):
    kind = s["kind"]
    if kind == "gemm":
        return gemm(s["A"], s["B"], s["C"], beta=s["beta"], path=s["path"])
    if kind == "gemm_i8":
        return gemm_i8(s["A"], s["B"], s["C"], beta=s["beta"])
    if kind == "fp8_packed":
        M, N, K, stream = s["M"], s["N"], s["K"], torch.cuda.current_stream().cuda_stream
        _native.check(_native.mg_fp8_pack("N", M, K, s["X"].data_ptr(), K, s["qx"].data_ptr(), s["sx"].data_ptr(),
                                          stream), "mg_fp8_pack")
        _native.check(_native.mg_gemm_fp8_packed(M, N, K, 1.0, s["qx"].data_ptr(), s["sx"].data_ptr(),
                                                 s["qw"].data_ptr(), s["sw"].data_ptr(), 0.0, s["Y"].data_ptr(), N,
                                                 stream), "mg_gemm_fp8_packed")
        return s["Y"]
    if kind == "train":
        Y = matmul(s["X"], s["W"], s["path"])
        dX, dW = torch.autograd.grad(Y, (s["X"], s["W"]), s["G"])
        return Y, dX, dW
    if kind == "batched":
        gemm_batched(s["problems"], path=s["path"])
        return s["C"]
    A, B, C = s["A"], s["B"], s["C"]
    _native.check(_native.mg_syr2k(0, s["uplo"], s["trans"], s["N"], s["K"], 1.0, A.data_ptr(), A.stride(0),
                                   B.data_ptr(), B.stride(0), s["beta"], C.data_ptr(), C.stride(0),
                                   s["workspace"].data_ptr(), s["bytes"], torch.cuda.current_stream().cuda_stream),
                  "mg_syr2k")
    return C


def work(case):
    kind = case["kind"]
    if kind == "batched":
        sizes = _batch_sizes(case)
        return {"bytes": sum(4 * (m * k + k * n + m * n) for m, n, k in sizes),
                "flops": sum(2 * m * n * k for m, n, k in sizes)}
    N, K = case["N"], case["K"]
    if kind == "syr2k":
        tri = N * (N + 1) // 2
        return {"bytes": 8 * N * K + 4 * tri * (2 if case["beta"] else 1), "flops": 4 * tri * K}
    M = case["M"]
    out = M * N * (2 if case.get("beta") else 1)
    if kind == "train":
        return {"bytes": 4 * (2 * (M * K + K * N) + 2 * M * N), "flops": 6 * M * N * K}
    if kind == "fp8_packed":
        return {"bytes": 4 * M * K + N * K + 4 * M * N, "flops": 2 * M * N * K}
    return {"bytes": (1 if kind == "gemm_i8" else 4) * (M * K + K * N) + 4 * out, "flops": 2 * M * N * K}


def exact(case, seed):
    s = prepare(case, seed)
    kind = case["kind"]
    if kind in ("gemm", "gemm_i8"):
        C = s["A"].double() @ s["B"].double()
        if case["beta"]:
            C += case["beta"] * s["C"].double()
        return C if kind == "gemm" else C.round().to(torch.int64).to(torch.int32)
    if kind == "fp8_packed":
        return s["X"].double() @ s["W"].double().t()
    if kind == "train":
        X, W, G = (s[k].detach().double() for k in "XWG")
        return X @ W, G @ W.t(), X.t() @ G
    if kind == "batched":
        C = torch.zeros_like(s["C"], dtype=torch.float64)
        for (a, b, c, _, _) in s["problems"]:
            at = c.storage_offset()
            C[at:at + c.numel()] = (a.double() @ b.double()).reshape(-1)
        return C
    X, Y, C = s["A"].double(), s["B"].double(), s["C"].double()
    P = X @ Y.t() if case["trans"] == "N" else X.t() @ Y
    full = P + P.t() + case["beta"] * C
    keep = torch.ones_like(C, dtype=torch.bool)
    return torch.where(keep.tril() if case["uplo"] == "L" else keep.triu(), full, C)
