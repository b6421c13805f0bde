"""The work a user of this library has it do, as cases that can be measured one by one.

What a program does with the library, over and over, is launch the kernel of one member of a configuration space
(opevo_kernel_launch: inside a search that is every trial, after a search it is the use of what was found) and compare an
output with a reference on the device (the parity gate of every trial).  Each case below is one such call.  A case names the
operator, its extents, the input type, the space and the member; the listed ones are the operators this repository
measures, each with a member that a search over 150 - 1000 trials ended on.  Kernels are compiled before the pass, as a
program that launches one does, and inputs follow the distributions of `paper_2006_05664_amd/synth.py`.
"""
from __future__ import annotations

import math
import random
from typing import Dict, List

import torch

import paper_2006_05664_amd as P

_DTYPE = {"f32": (P.OPEVO_F32, torch.float32), "bf16": (P.OPEVO_BF16, torch.bfloat16), "f16": (P.OPEVO_F16, torch.float16)}
_KIND = {"matmul": P.OPEVO_MATMUL, "bmm": P.OPEVO_BMM, "bmm_ta": P.OPEVO_BMM_TA, "conv2d": P.OPEVO_CONV2D}
_SPACE = {"TILE2": P.OPEVO_TILE2, "TILE4": P.OPEVO_TILE4, "TILE4A": P.OPEVO_TILE4A, "TILE4C": P.OPEVO_TILE4C, "TILE4L": P.OPEVO_TILE4L}


def _op_case(kind: str, dims, dtype: str, space: str, cfg, name: str = "") -> Dict:
    case = {"name": name} if name else {}
    case.update(kind=kind, dims=",".join(map(str, dims)), dtype=dtype, space=space, cfg=",".join(map(str, cfg)))
    return case


def _ints(text: str) -> List[int]:
    return [int(x) for x in text.split(",")]


def listed() -> List[Dict]:
    return [
        # the smallest call: the 64^3 fp32 MatMul of the two-level space, all launch and latency
        _op_case("matmul", (64, 64, 64), "f32", "TILE2", (32, 2, 32, 2, 1, 64), "mm64_f32"),
        # an ordinary projection (512 x 1024 x 1024) in 16 bits
        _op_case("matmul", (512, 1024, 1024), "bf16", "TILE4", (8, 2, 8, 4, 16, 2, 4, 8, 16, 64, 1), "mm1_bf16"),
        # extents that are no multiples of the matrix atoms: 1000 = 8 * 125 rows, columns and reduction steps
        _op_case("matmul", (1000, 1000, 1000), "bf16", "TILE4", (50, 4, 1, 5, 10, 5, 20, 1, 10, 100, 1), "mm1000_bf16"),
        # the largest MatMul, the one the matrix pipes bound
        _op_case("matmul", (8192, 8192, 8192), "bf16", "TILE4A", (32, 2, 32, 4, 32, 4, 32, 2, 64, 128, 1, 1), "mm8192_bf16"),
        # the paper's precision: fp32 inputs on fp32 matrix atoms, 512 x 4096 x 1024
        _op_case("matmul", (512, 4096, 1024), "f32", "TILE4", (8, 2, 16, 2, 64, 2, 32, 1, 16, 64, 1), "mm2_f32"),
        # attention scores: a batch of 128 products of 128 x 128 x 64
        _op_case("bmm", (128, 128, 128, 64), "bf16", "TILE4", (128, 1, 1, 4, 8, 4, 2, 1, 32, 2, 2, 32, 1), "bmm_attn_bf16"),
        # a large batch with the first operand stored transposed, fp16
        _op_case("bmm_ta", (960, 128, 64, 128), "f16", "TILE4", (480, 2, 1, 2, 32, 2, 1, 2, 8, 4, 4, 32, 1), "bmm2_f16"),
        # one image through a 3x3 convolution, 64 -> 64 channels at 56 x 56: inference at batch 1, launch-bound
        _op_case("conv2d", (1, 64, 56, 56, 64, 3, 3, 1, 1), "bf16", "TILE4L",
                 (1, 1, 4, 2, 4, 2, 7, 2, 4, 1, 7, 2, 4, 1, 1, 64, 0, 2, 2), "conv56_bf16"),
        # a batch of 32 through a 3x3 convolution, 256 -> 256 channels at 14 x 14
        _op_case("conv2d", (32, 256, 14, 14, 256, 3, 3, 1, 1), "bf16", "TILE4L",
                 (32, 1, 8, 1, 8, 4, 1, 7, 2, 1, 1, 14, 1, 1, 8, 32, 0, 2, 1), "conv14_bf16"),
        # AlexNet's second convolution at batch 512: 5x5 taps, images of odd width (27 x 27)
        _op_case("conv2d", (512, 64, 27, 27, 192, 5, 5, 1, 2), "bf16", "TILE4L",
                 (256, 2, 3, 1, 32, 2, 3, 3, 1, 3, 1, 9, 1, 3, 16, 4, 0, 2, 1), "c2_bf16"),
        # AlexNet's first convolution at batch 512: 3 input channels, 11x11 taps, stride 4
        _op_case("conv2d", (512, 3, 227, 227, 64, 11, 11, 4, 0), "bf16", "TILE4C",
                 (128, 4, 1, 4, 8, 2, 55, 1, 1, 1, 1, 1, 5, 11, 1, 33, 11, 0, 0), "c1_bf16"),
        # the parity gate over an output the size of AlexNet's second convolution's
        {"name": "gate_whole", "kind": "gate", "rows": 0, "total_rows": 512 * 192, "row_len": 27 * 27},
    ]


# ------------------------------------------------------------------ members for drawn operators
def _divisors(n: int) -> List[int]:
    return [d for d in range(1, n + 1) if n % d == 0]


def _wave_tile(n: int, cap: int) -> int:
    """The divisor of n, at most cap, that fills whole 16-row atoms best (larger first among equals)."""
    return max((d for d in _divisors(n) if d <= cap), key=lambda d: (round(d / (16 * math.ceil(d / 16)), 2) if d >= 8 else 0.0, d))


def _split(n: int, cap: int, waves: int) -> List[int]:
    t = _wave_tile(n, cap)
    w = max(d for d in _divisors(n // t) if d <= waves)
    return [n // (t * w), w, 1, t]


def _slab(n: int, cap: int) -> List[int]:
    d = max(_divisors(n), key=lambda d: (d <= cap, (d % 32 == 0) + (d % 16 == 0), d))
    return [n // d, d]


def _gemm_member(kind: str, dims, dtype: str):
    batch, (M, N, K) = (1, dims) if kind == "matmul" else (dims[0], dims[1:])
    cap = 32
    if dtype != "f32" and batch * M * N >= 256 * 128 * 128:
        cap = 64            # enough tiles for the chip with 128 x 128 workgroups
    return ([] if kind == "matmul" else [batch, 1]) + _split(M, cap, 2) + _split(N, cap, 2) + _slab(K, 64) + [1]


def _conv_member(dims, rng_flag: int):
    B, cin, H, W, cout, hk, wk, stride, pad = dims
    ho, wo = (H + 2 * pad - hk) // stride + 1, (W + 2 * pad - wk) // stride + 1
    bw = max(d for d in _divisors(wo) if d <= 32)
    bh = max(d for d in _divisors(ho) if d * bw <= 224)
    hw = min((d for d in _divisors(bh) if d <= 8), key=lambda d: (abs(math.log(bh // d * bw / 40.0)), d))
    box = [ho // bh, hw, bh // hw, 1, wo // bw, 1, bw, 1]
    if cin % 16:            # no patch member: the gather, a kernel row (or a whole small kernel) at a time
        bk = hk * wk if hk * wk <= 32 else wk
        return "TILE4C", [B, 1] + [cout // 64, 4, 1, 16] + box + [1, cin * hk * wk // bk, bk, 0, 0]
    wm = 2 if cout % 64 == 0 else 1
    return "TILE4L", [B, 1] + [cout // (32 * wm), wm, 1, 32] + box + [cin // 16, 16, rng_flag, 2, 0]


def _log(rng: random.Random, lo: float, hi: float) -> float:
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _extent(rng: random.Random, lo: int, hi: int, ragged: bool) -> int:
    """An extent made of whole tiles: tiles of 32 or 64, or (ragged) of 20 to 60, odd ones among them."""
    t = rng.choice((20, 21, 24, 25, 27, 28, 30, 33, 35, 36, 40, 45, 50, 55, 60) if ragged else (32, 64))
    return t * max(1, round(_log(rng, lo, hi) / t))


def draw(rng: random.Random) -> Dict:
    family = rng.choice(("tiny", "matmul", "matmul", "matmul", "bmm", "bmm", "conv", "conv", "conv", "gate"))
    if family == "tiny":
        M, N, K = (rng.choice((16, 24, 30, 32, 48, 50, 64, 72, 96, 100, 128)) for _ in range(3))
        return _op_case("matmul", (M, N, K), "f32", "TILE2", (M // 2, 2, N // 2, 2, 1, K))
    if family in ("matmul", "bmm"):
        dtype = rng.choice(("bf16", "f16", "f32"))
        ragged = dtype != "f32" and rng.random() < 0.5
        kind = "matmul" if family == "matmul" else rng.choice(("bmm", "bmm_ta"))
        most = 1e10 if ragged else 5e10 if dtype == "f32" else 1e12       # flops: no more time than the largest listed case
        while True:
            if kind == "matmul":
                dims = [_extent(rng, 64, 8192, ragged) for _ in range(3)]
            else:
                dims = [round(_log(rng, 8, 1000))] + [_extent(rng, 32, 256, ragged) for _ in range(3)]
            if 2.0 * math.prod(dims) <= most:
                return _op_case(kind, dims, dtype, "TILE4", _gemm_member(kind, dims, dtype))
    if family == "conv":
        cin = rng.choice((1, 3, 16, 32, 48, 64, 96, 128, 256))
        if cin < 16:
            k, stride, size = rng.choice((3, 5, 7, 11)), rng.choice((1, 2, 4)), rng.choice((28, 56, 64, 112, 113, 224, 227))
        else:
            k, stride, size = rng.choice((1, 3, 3, 5)), rng.choice((1, 1, 1, 2)), rng.choice((7, 13, 14, 27, 28, 55, 56))
        cout = rng.choice((64, 128, 192)) if cin < 16 else rng.choice((32, 64, 96, 128, 192, 256))
        pad = 0 if stride == 4 else k // 2
        out = (size + 2 * pad - k) // stride + 1
        per_image = 2.0 * cout * out * out * cin * k * k
        top = max(1.0, min(256.0, 1e11 / per_image, 3e8 / (cout * out * out * 4)))
        dims = [max(1, round(_log(rng, 1, top))), cin, size, size, cout, k, k, stride, pad]
        space, cfg = _conv_member(dims, rng.choice((0, 1)))
        return _op_case("conv2d", dims, rng.choice(("bf16", "f16")), space, cfg)
    # the gate over a whole output, or over a sample of its rows
    row_len = round(_log(rng, 64, 8192))
    total = max(1, round(_log(rng, 4096, 6e7) / row_len))
    return {"kind": "gate", "rows": rng.choice((0, max(1, total // 4))), "total_rows": total, "row_len": row_len}


# ------------------------------------------------------------------ inputs and the pass
class _Kernel:
    """An instantiated member, destroyed with its owner."""

    def __init__(self, case: Dict):
        self.handle = self.op = None
        self.op = P.opevo_op_create(_KIND[case["kind"]], _ints(case["dims"]), _DTYPE[case["dtype"]][0])
        self.handle, _ = P.opevo_kernel_build(self.op, _SPACE[case["space"]], _ints(case["cfg"]))
        self.c_elems = P.opevo_op_sizes(self.op)[2]

    def __del__(self):
        if self.handle is not None:
            P.opevo_kernel_destroy(self.handle)
        if self.op is not None:
            P.opevo_op_destroy(self.op)


def _operands(case: Dict, seed: int):
    """First and second operand in the order the kernels take them."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    td, dims = _DTYPE[case["dtype"]][1], _ints(case["dims"])

    def normal(*shape, scale=1.0):
        return torch.randn(shape, generator=g, device="cuda").mul_(scale).to(td)

    if case["kind"] == "matmul":
        M, N, K = dims
        return normal(M, K, scale=K ** -0.5), normal(K, N, scale=K ** -0.5)
    if case["kind"] == "bmm":
        b, M, N, K = dims
        return normal(b, M, K), normal(b, K, N)
    if case["kind"] == "bmm_ta":
        b, M, N, K = dims
        return normal(b, K, M), normal(b, K, N)
    B, cin, H, W, cout, hk, wk = dims[:7]
    return normal(cout, cin, hk, wk, scale=0.05), torch.rand((B, cin, H, W), generator=g, device="cuda").to(td)


def _out_shape(case: Dict):
    d = _ints(case["dims"])
    if case["kind"] == "matmul":
        return d[0], d[1]
    if case["kind"] in ("bmm", "bmm_ta"):
        return d[0], d[1], d[2]
    B, _, H, W, cout, hk, wk, stride, pad = d
    return B, cout, (H + 2 * pad - hk) // stride + 1, (W + 2 * pad - wk) // stride + 1


def _gate_inputs(case: Dict, seed: int):
    """An fp32 output that differs from its reference by what an fp32 summation order gives."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    total, row_len, rows = case["total_rows"], case["row_len"], case["rows"]
    c = torch.randn((total, row_len), generator=g, device="cuda")
    index = None
    ref = c
    if rows:
        index = torch.randperm(total, generator=g, device="cuda")[:rows].sort().values.to(torch.int32)
        ref = c[index.long()]
    ref = ref + 1e-5 * torch.randn(ref.shape, generator=g, device="cuda")
    return c, ref, index


def prepare(case: Dict, seed: int) -> Dict:
    stream = torch.cuda.current_stream().cuda_stream
    if case["kind"] == "gate":
        c, ref, index = _gate_inputs(case, seed)
        return {"c": c, "ref": ref, "index": index, "row_len": case["row_len"], "stream": stream}
    a, b = _operands(case, seed)
    return {"kernel": _Kernel(case), "a": a, "b": b, "c": torch.empty(_out_shape(case), device="cuda"), "stream": stream}


def run(state: Dict):
    if "ref" in state:
        c, ref, index = state["c"], state["ref"], state["index"]
        if index is None:
            return P.opevo_compare_f32(c.data_ptr(), ref.data_ptr(), ref.numel(), state["stream"])
        return P.opevo_compare_rows_f32(c.data_ptr(), ref.data_ptr(), index.data_ptr(), index.numel(), state["row_len"], state["stream"])
    P.opevo_kernel_launch(state["kernel"].handle, state["a"].data_ptr(), state["b"].data_ptr(), state["c"].data_ptr(), state["stream"])
    return state["c"]


def work(case: Dict) -> Dict:
    if case["kind"] == "gate":
        n = (case["rows"] or case["total_rows"]) * case["row_len"]
        return {"bytes": 8.0 * n, "flops": 8.0 * n}
    op = P.opevo_op_create(_KIND[case["kind"]], _ints(case["dims"]), _DTYPE[case["dtype"]][0])
    try:
        return {"bytes": P.opevo_op_bytes(op), "flops": P.opevo_op_flops(op)}
    finally:
        P.opevo_op_destroy(op)


def tolerance(case: Dict) -> Dict:
    # the gate sums in 64 bits; the operators in 32, over at most a few thousand products: against 64 bits they were seen
    # between 4e-8 and 6e-7 (most with fp32 inputs), and a longer sum in another order shows a few times that
    return {"rel": 1e-10} if case["kind"] == "gate" else {"rel": 1e-5}


def exact(case: Dict, seed: int):
    if case["kind"] == "gate":
        c, ref, index = _gate_inputs(case, seed)
        if index is not None:
            c = c[index.long()]
        c, ref = c.double(), ref.double()
        d = c - ref
        return float((d.abs() / (ref.abs() + 1.0)).max()), float(d.norm() / ref.norm())
    a, b = _operands(case, seed)
    if case["kind"] == "matmul":
        return a.double() @ b.double()
    if case["kind"] in ("bmm", "bmm_ta"):
        a = a.double()
        return torch.bmm(a.transpose(1, 2).contiguous() if case["kind"] == "bmm_ta" else a, b.double())
    shape, dims = _out_shape(case), _ints(case["dims"])
    w = a.double().reshape(a.shape[0], -1)
    out = torch.empty(shape, dtype=torch.float64, device="cuda")
    step = max(1, int(2e8 / (w.shape[1] * shape[2] * shape[3])))
    for i in range(0, shape[0], step):       # a few images at a time: every output pixel's taps side by side, then one product
        cols = torch.nn.functional.unfold(b[i:i + step].double(), tuple(dims[5:7]), padding=dims[8], stride=dims[7])
        n = cols.shape[0]
        flat = cols.permute(1, 0, 2).reshape(w.shape[1], -1)
        out[i:i + n] = (w @ flat).reshape(shape[1], n, shape[2], shape[3]).permute(1, 0, 2, 3)
    return out
