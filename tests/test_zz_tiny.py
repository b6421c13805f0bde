"""Scalar-template tiles of a few outputs whose lanes share an output: reductions shorter than the lanes that share, no
multiple of them, one more than the unrolled eight steps, several batches, partitions and slabs, the deadline honoured
without a barrier.  fp32 sums of at most 4096 products: 1e-5 is 80 roundings of the result."""
import numpy as np
import pytest

import paper_2006_05664_amd as P
from paper_2006_05664_amd import synth

pytestmark = pytest.mark.gpu

CASES = [   # label, kind, dims, dtype, space, configuration
    ("2x2, 16 lanes, 64 steps", P.OPEVO_MATMUL, (64, 64, 64), "f32", P.OPEVO_TILE2, [32, 2, 32, 2, 1, 64]),
    ("one output, 64 lanes, 65 steps", P.OPEVO_MATMUL, (3, 5, 65), "f32", P.OPEVO_TILE2, [3, 1, 5, 1, 5, 13]),
    ("one output, 576 steps and 7 more", P.OPEVO_MATMUL, (3, 5, 583), "f32", P.OPEVO_TILE2, [3, 1, 5, 1, 53, 11]),
    ("more lanes than steps", P.OPEVO_MATMUL, (4, 6, 5), "f32", P.OPEVO_TILE2, [2, 2, 3, 2, 1, 5]),
    ("4x4, 4 lanes, slabs of one", P.OPEVO_MATMUL, (16, 12, 50), "f32", P.OPEVO_TILE2, [4, 4, 3, 4, 50, 1]),
    ("long reduction", P.OPEVO_MATMUL, (4, 4, 4096), "f32", P.OPEVO_TILE2, [2, 2, 2, 2, 64, 64]),
    ("bf16, four waves", P.OPEVO_MATMUL, (32, 48, 96), "bf16", P.OPEVO_TILE4, [8, 2, 2, 1, 24, 2, 1, 1, 3, 32, 1]),
    ("fp16 batches, two per workgroup", P.OPEVO_BMM, (6, 8, 16, 33), "f16", P.OPEVO_TILE4, [3, 2, 4, 1, 1, 2, 4, 1, 1, 4, 3, 11, 1]),
    ("reduction over 4 workgroups", P.OPEVO_MATMUL, (16, 16, 96), "f32", P.OPEVO_TILE4K, [8, 1, 1, 2, 8, 1, 1, 2, 4, 3, 8, 1]),
]


@pytest.mark.parametrize("label,kind,dims,dtype,variant,cfg", CASES, ids=[c[0] for c in CASES])
def test_results_match_the_oracle(label, kind, dims, dtype, variant, cfg):
    import torch
    from oracle import tensor as T
    a, b = (synth.matmul_inputs if kind == P.OPEVO_MATMUL else synth.bmm_inputs)(*dims, dtype, 5)
    want = (T.matmul if kind == P.OPEVO_MATMUL else T.bmm)(a, b)
    op = P.opevo_op_create(kind, dims, synth.DTYPE_CODE[dtype])
    assert P.opevo_kernel_plan(op, variant, cfg).path == 0
    da, db = synth.to_device(a, dtype), synth.to_device(b, dtype)
    dc = torch.full((want.size,), float("nan"), device="cuda:0")
    kernel, _ = P.opevo_kernel_build(op, variant, cfg)
    stream = torch.cuda.current_stream().cuda_stream
    for _ in range(2):
        P.opevo_kernel_launch(kernel, da.data_ptr(), db.data_ptr(), dc.data_ptr(), stream)
    torch.cuda.synchronize()
    got = dc.cpu().numpy().astype(np.float64)
    assert np.all(np.isfinite(got)) and np.linalg.norm(got - want.ravel()) <= 1e-5 * np.linalg.norm(want), label
    # a deadline that cannot be met is reported, and one that can is not
    ms, _ = P.opevo_kernel_time(kernel, da.data_ptr(), db.data_ptr(), dc.data_ptr(), stream, timeout_ms=1000.0, warmup_ms=0.0)
    assert ms > 0
    P.opevo_kernel_destroy(kernel)


def test_a_tiny_tile_honours_the_deadline():
    import torch
    op = P.opevo_op_create(P.OPEVO_MATMUL, (2, 2, 1 << 22), P.OPEVO_F32)     # one workgroup, 2^18 steps per lane: some ten ms
    cfg = [1, 2, 1, 2, 1 << 11, 1 << 11]
    a, b = torch.ones(2 << 22, device="cuda"), torch.ones(2 << 22, device="cuda")
    c = torch.empty(4, device="cuda")
    kernel, _ = P.opevo_kernel_build(op, P.OPEVO_TILE2, cfg)
    stream = torch.cuda.current_stream().cuda_stream
    with pytest.raises(P.OpevoError) as e:
        P.opevo_kernel_time(kernel, a.data_ptr(), b.data_ptr(), c.data_ptr(), stream, timeout_ms=0.5)
    assert e.value.status == P.OPEVO_E_INVALID and "deadline" in e.value.message
    P.opevo_kernel_launch(kernel, a.data_ptr(), b.data_ptr(), c.data_ptr(), stream)      # a launch has none
    torch.cuda.synchronize()
    assert torch.all(c == float(1 << 22))
    P.opevo_kernel_destroy(kernel)


def test_a_deadline_holds_where_a_lane_has_fewer_than_eight_steps():
    import torch
    op = P.opevo_op_create(P.OPEVO_MATMUL, (4096, 4096, 16), P.OPEVO_F32)     # 2^24 workgroups of one output, one step per lane: some ten ms
    a, b = torch.ones(4096 * 16, device="cuda"), torch.ones(4096 * 16, device="cuda")
    c = torch.empty(4096 * 4096, device="cuda")
    kernel, _ = P.opevo_kernel_build(op, P.OPEVO_TILE2, [4096, 1, 4096, 1, 1, 16])
    stream = torch.cuda.current_stream().cuda_stream
    with pytest.raises(P.OpevoError) as e:
        P.opevo_kernel_time(kernel, a.data_ptr(), b.data_ptr(), c.data_ptr(), stream, timeout_ms=0.5)
    assert e.value.status == P.OPEVO_E_INVALID and "deadline" in e.value.message
    P.opevo_kernel_launch(kernel, a.data_ptr(), b.data_ptr(), c.data_ptr(), stream)      # a launch has none
    torch.cuda.synchronize()
    assert torch.all(c == 16.0)
    P.opevo_kernel_destroy(kernel)
