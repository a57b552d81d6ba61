"""Representative calls of the library, for timing one build against another.

Each case is one call of a public entry point of ``paper_2505_18574_amd.ops`` on buffers that a caller keeps in
device memory: the accelerator-sized int8 layers whose launch lasts microseconds, the layers and products that fill
the chip, sizes that are a multiple of nothing, and the two fp32 streams.  ``listed()`` names a dozen of them and
``draw(rng)`` gives further ones of the same kinds and ranges; ``prepare`` makes a case's inputs on the GPU,
``run`` is the call, ``work`` what it cannot do without and ``tolerance`` how far two correct results may differ.
"""
from __future__ import annotations

import math

import torch

from paper_2505_18574_amd import ops


# ----------------------------------------------------------------------------
# cases
# ----------------------------------------------------------------------------
def _gemm_i8(M, N, K, out="i8", trans_a=False, trans_b=False):
    """out: "i8" = the output stage with a bias row and ReLU, "i32" = the raw accumulator."""
    return {"kind": "gemm_i8", "M": M, "N": N, "K": K, "out": out, "trans_a": trans_a, "trans_b": trans_b}


def _conv_i8(Nb, H, W, Cin, Cout, k, stride, pad):
    return {"kind": "conv_i8", "Nb": Nb, "H": H, "W": W, "Cin": Cin, "Cout": Cout, "k": k, "stride": stride, "pad": pad}


def _gemm_bf16(M, N, K):
    return {"kind": "gemm_bf16", "M": M, "N": N, "K": K}


def _batched(batch, n, matvec=True):
    return {"kind": "batched_f32", "batch": batch, "n": n, "matvec": matvec}


def _tinympc(batch, nx, nu, horizon, trajectory=True):
    return {"kind": "tinympc", "batch": batch, "nx": nx, "nu": nu, "horizon": horizon, "trajectory": trajectory}


def listed():
    return [
        # the smallest call: the 256^3 tile of an accelerator-sized layer, all launch and latency
        {"name": "gemm_i8_256", **_gemm_i8(256, 256, 256)},
        # a late layer on a 7 x 7 image: few rows against 9 MB of weights, cut along K through a workspace
        {"name": "gemm_i8_49x2048x4608", **_gemm_i8(49, 2048, 4608)},
        # a classifier-sized product whose rows are not whole 16-byte chunks
        {"name": "gemm_i8_1000", **_gemm_i8(1000, 1000, 1000)},
        # a middle layer with its weights stored output-channel first (N x K)
        {"name": "gemm_i8_t_784x512x1152", **_gemm_i8(784, 512, 1152, trans_b=True)},
        # the largest int8 product, bound by the matrix units
        {"name": "gemm_i8_8192", **_gemm_i8(8192, 8192, 8192)},
        # ResNet-50 convolutions: a 3 x 3 layer at inference batch, ...
        {"name": "conv_i8_56x56_64to64", **_conv_i8(8, 56, 56, 64, 64, 3, 1, 1)},
        # ... the first layer on a three-channel image, ...
        {"name": "conv_i8_224x224_3to64_s2", **_conv_i8(8, 224, 224, 3, 64, 7, 2, 3)},
        # ... and a down-sampling layer at a throughput batch
        {"name": "conv_i8_28x28_128to256_s2_b256", **_conv_i8(256, 28, 28, 128, 256, 3, 2, 1)},
        # the large bf16 product of the GPU study
        {"name": "gemm_bf16_4096", **_gemm_bf16(4096, 4096, 4096)},
        # a bf16 product with odd sizes in every dimension
        {"name": "gemm_bf16_1023x1537x1021", **_gemm_bf16(1023, 1537, 1021)},
        # fine-grained linear algebra: a stream of 12 x 12 products with a mat-vec and an add
        {"name": "batched_f32_262144x12", **_batched(262144, 12)},
        # a forward pass of the controller over as many problems
        {"name": "tinympc_262144x12x4x5", **_tinympc(262144, 12, 4, 5)},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _size(rng, lo, hi, whole):
    """A size of [lo, hi], spread over its logarithm and rounded to a multiple of `whole` (of 1: as it falls)."""
    return min(hi, max(whole, (_log_int(rng, lo, hi) + whole // 2) // whole * whole))


def draw(rng):
    kind = rng.choices(["gemm_i8", "conv_i8", "gemm_bf16", "batched_f32", "tinympc"], [8, 5, 5, 4, 3])[0]
    if kind in ("gemm_i8", "gemm_bf16"):
        # half of the products in whole 64s, a quarter in whole 4s, a quarter as they fall
        whole = rng.choices([64, 4, 1], [2, 1, 1])[0]
        # up to the largest listed product of the type; sizes that are a multiple of nothing stay below a quarter of
        # its edge
        cap = (8192 if kind == "gemm_i8" else 4096) // (1 if whole == 64 else 4)
        M, N, K = _size(rng, 16, cap, 1 if whole == 1 else 4), _size(rng, 16, cap, whole), _size(rng, 16, cap, whole)
        if kind == "gemm_bf16":
            return _gemm_bf16(M, N, K)
        form = rng.choices(["plain", "i32", "ta", "tb", "tab"], [6, 1, 1, 2, 1])[0]
        return _gemm_i8(M, N, K, "i32" if form == "i32" else "i8", form in ("ta", "tab"), form in ("tb", "tab"))
    if kind == "conv_i8":
        # image edge and channels trade off as in a ResNet-50; one in four starts from an image of few channels and
        # one in eight has channel counts that are a multiple of nothing
        form = rng.choices(["layer", "image", "odd"], [5, 2, 1])[0]
        k = rng.choice([1, 3, 3, 5, 7])
        stride = rng.choice([1, 1, 2])
        if form == "image":
            edge, cin, cout, nb = _log_int(rng, 32, 256), rng.choice([1, 3, 3, 4]), 16 * rng.randint(1, 6), _log_int(rng, 1, 32)
        elif form == "layer":
            edge, nb = _log_int(rng, 7, 56), _log_int(rng, 1, 64)
            cin, cout = 16 * _log_int(rng, 1, 32), 16 * _log_int(rng, 1, 32)
        else:
            edge, cin, cout, nb = _log_int(rng, 7, 56), rng.randint(2, 60), rng.randint(2, 60), _log_int(rng, 1, 8)
        return _conv_i8(nb, edge, edge, cin, cout, k, stride, k // 2)
    if kind == "batched_f32":
        n = rng.choice([12, rng.randint(2, 16), rng.randint(2, 16)])
        return _batched(_log_int(rng, 64, 262144), n, rng.random() < 0.75)
    nx, nu = (12, 4) if rng.random() < 0.5 else (rng.randint(2, 16), rng.randint(1, 8))
    return _tinympc(_log_int(rng, 64, 262144), nx, nu, rng.choice([5, 5, rng.randint(1, 10)]), rng.random() < 0.75)


# ----------------------------------------------------------------------------
# inputs, as a caller holds them on the GPU
# ----------------------------------------------------------------------------
def _generator(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _i8(g, *shape):
    return torch.randint(-128, 128, shape, dtype=torch.int8, device="cuda", generator=g)


def _bias(g, n):
    return torch.randint(-(1 << 15), 1 << 15, (n,), dtype=torch.int32, device="cuda", generator=g)


def _unit(g, *shape):
    return torch.rand(shape, dtype=torch.float32, device="cuda", generator=g) * 2 - 1


def _shift(K):
    """A scale-down that leaves the sums of K products of uniform int8 with a deviation of some 45 before the clamp,
    as a calibrated layer has it."""
    return max(1, round(math.log2(math.sqrt(K) * 5461 / 45)))


def _workspace(nbytes):
    return torch.empty(nbytes, dtype=torch.uint8, device="cuda") if nbytes else None


def _conv_out(case):
    return tuple((case[e] + 2 * case["pad"] - case["k"]) // case["stride"] + 1 for e in ("H", "W"))


def prepare(case, seed):
    g = _generator(seed)
    s = dict(case)
    kind = case["kind"]
    if kind == "gemm_i8":
        M, N, K = case["M"], case["N"], case["K"]
        s["A"] = _i8(g, K, M) if case["trans_a"] else _i8(g, M, K)
        s["B"] = _i8(g, N, K) if case["trans_b"] else _i8(g, K, N)
        s["bias"], s["shift"] = _bias(g, N), _shift(K)
        s["C"] = torch.empty((M, N), dtype=torch.int32 if case["out"] == "i32" else torch.int8, device="cuda")
        s["workspace"] = _workspace(ops.ac_gemm_i8_workspace_bytes(M, N, K))
    elif kind == "conv_i8":
        k, cin, cout = case["k"], case["Cin"], case["Cout"]
        oh, ow = _conv_out(case)
        s["x"], s["w"] = _i8(g, case["Nb"], case["H"], case["W"], cin), _i8(g, k, k, cin, cout)
        s["bias"], s["shift"] = _bias(g, cout), _shift(k * k * cin)
        s["out"] = torch.empty((case["Nb"], oh, ow, cout), dtype=torch.int8, device="cuda")
        s["workspace"] = _workspace(ops.ac_gemm_i8_workspace_bytes(case["Nb"] * oh * ow, cout, k * k * cin))
    elif kind == "gemm_bf16":
        M, N, K = case["M"], case["N"], case["K"]
        s["A"] = torch.randn((M, K), dtype=torch.float32, device="cuda", generator=g).to(torch.bfloat16)
        s["B"] = torch.randn((K, N), dtype=torch.float32, device="cuda", generator=g).to(torch.bfloat16)
        s["C"] = torch.empty((M, N), dtype=torch.float32, device="cuda")
        s["workspace"] = _workspace(ops.ac_gemm_bf16_workspace_bytes(M, N, K))
    elif kind == "batched_f32":
        b, n = case["batch"], case["n"]
        s["A"], s["B"] = _unit(g, b, n, n), _unit(g, b, n, n)
        s["x"], s["d"] = (_unit(g, b, n), _unit(g, b, n)) if case["matvec"] else (None, None)
        s["C"] = torch.empty((b, n, n), dtype=torch.float32, device="cuda")
        s["y"] = torch.empty((b, n), dtype=torch.float32, device="cuda") if case["matvec"] else None
    else:
        b, nx, nu, h = case["batch"], case["nx"], case["nu"], case["horizon"]
        # a loop that neither dies out nor blows up over the horizon
        s["Adyn"] = _unit(g, nx, nx) / max(1.0, 0.6 * math.sqrt(nx))
        s["Bdyn"], s["Kinf"] = _unit(g, nx, nu) / math.sqrt(nx), _unit(g, nu, nx) / math.sqrt(nx)
        s["x0"], s["d"] = _unit(g, b, nx), _unit(g, b, h, nu)
        s["u"] = torch.empty((b, h, nu), dtype=torch.float32, device="cuda")
        s["x_out"] = torch.empty((b, h + 1, nx), dtype=torch.float32, device="cuda") if case["trajectory"] else None
    return s


def run(s):
    kind = s["kind"]
    if kind == "gemm_i8":
        if s["out"] == "i32":
            return ops.ac_gemm_i8_acc32(s["A"], s["B"], s["bias"], s["C"])
        if s["trans_a"] or s["trans_b"]:
            return ops.ac_gemm_i8_t(s["A"], s["B"], s["bias"], s["C"], s["shift"], ops.AC_ACT_RELU, trans_a=s["trans_a"], trans_b=s["trans_b"])
        return ops.ac_gemm_i8(s["A"], s["B"], s["bias"], s["C"], s["shift"], ops.AC_ACT_RELU, workspace=s["workspace"])
    if kind == "conv_i8":
        return ops.ac_conv2d_i8(s["x"], s["w"], s["bias"], s["out"], s["stride"], s["pad"], s["shift"], ops.AC_ACT_RELU, workspace=s["workspace"])
    if kind == "gemm_bf16":
        return ops.ac_gemm_bf16_ws(s["A"], s["B"], s["C"], workspace=s["workspace"])
    if kind == "batched_f32":
        C, y = ops.ac_batched_gemm_f32(s["A"], s["B"], s["C"], s["x"], s["d"], s["y"])
        return (C, y) if y is not None else C
    u, x = ops.ac_tinympc_forward_f32(s["Adyn"], s["Bdyn"], s["Kinf"], s["x0"], s["d"], s["u"], s["x_out"])
    return (u, x) if x is not None else u


# ----------------------------------------------------------------------------
# what a pass cannot do without, and how far two correct results may differ
# ----------------------------------------------------------------------------
def work(case):
    kind = case["kind"]
    if kind in ("gemm_i8", "gemm_bf16"):
        M, N, K = case["M"], case["N"], case["K"]
        if kind == "gemm_bf16":
            nbytes = 2 * (M * K + K * N) + 4 * M * N
        else:
            nbytes = M * K + K * N + 4 * N + M * N * (4 if case["out"] == "i32" else 1)
        return {"bytes": nbytes, "flops": 2 * M * N * K}
    if kind == "conv_i8":
        oh, ow = _conv_out(case)
        m, n, k = case["Nb"] * oh * ow, case["Cout"], case["k"] ** 2 * case["Cin"]
        return {"bytes": case["Nb"] * case["H"] * case["W"] * case["Cin"] + k * n + 4 * n + m * n, "flops": 2 * m * n * k}
    if kind == "batched_f32":
        b, n = case["batch"], case["n"]
        vec = 3 * n if case["matvec"] else 0
        return {"bytes": 4 * b * (3 * n * n + vec), "flops": b * (2 * n ** 3 + (2 * n * n + n if case["matvec"] else 0))}
    b, nx, nu, h = case["batch"], case["nx"], case["nu"], case["horizon"]
    floats = nx + 2 * h * nu + ((h + 1) * nx if case["trajectory"] else 0)
    steps = h if case["trajectory"] else h - 1  # the state after the last control is only computed for the trajectory
    return {"bytes": 4 * b * floats, "flops": b * (h * (2 * nx * nu + nu) + steps * 2 * nx * (nx + nu))}


def tolerance(case):
    if case["kind"] in ("gemm_i8", "conv_i8"):
        return "exact"
    # fp32 sums of exact bf16 products (4e-7 from float64 at K = 4096) and of fp32 products (up to 1.3e-7), four
    # times that: the sums may run in another order
    if case["kind"] == "gemm_bf16":
        return {"rel": 1.6e-6}
    return {"rel": 6e-7}
