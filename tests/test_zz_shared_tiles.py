"""Conv2d members with an LDS-resident patch whose workgroups have one or two waves: the waves that share a wave tile although
the member asks for none -- which members get how many, and their results at the edges of the rule."""
import numpy as np
import pytest

import paper_2006_05664_amd as P
from paper_2006_05664_amd import synth

CASES = [   # label, dims, dtype, waves (M, N), waves per tile, workgroups at least and at most, configuration
    ("one wave, 9 steps", (2, 16, 9, 9, 32, 3, 3, 1, 1), "bf16", (1, 1), 4, (1, 256), [1, 2, 1, 16, 1, 2, 1, 1, 9, 1, 1, 1, 1, 9, 1, 16, 0, 2, 0]),
    ("one wave, two slabs in flight", (3, 32, 13, 13, 64, 5, 5, 1, 2), "f16", (1, 1), 4, (1, 256), [1, 3, 1, 1, 1, 64, 13, 1, 1, 1, 1, 1, 1, 13, 8, 4, 1, 2, 0]),
    ("one wave, 16 x 16 atoms", (3, 32, 13, 13, 64, 5, 5, 1, 2), "bf16", (1, 1), 4, (1, 256), [3, 1, 2, 1, 1, 32, 1, 1, 1, 13, 13, 1, 1, 1, 1, 32, 0, 2, 0]),
    ("two waves along the channels", (3, 32, 13, 13, 64, 5, 5, 1, 2), "bf16", (2, 1), 2, (1, 512), [3, 1, 1, 4, 1, 16, 1, 1, 13, 1, 1, 1, 13, 1, 2, 16, 0, 2, 0]),
    ("two waves along the pixels", (30, 16, 14, 14, 64, 3, 3, 1, 1), "f16", (1, 2), 2, (1, 512), [3, 10, 1, 1, 1, 64, 7, 2, 1, 1, 1, 1, 14, 1, 4, 4, 1, 2, 0]),
    ("one wave, 280 workgroups", (30, 16, 14, 14, 64, 3, 3, 1, 1), "bf16", (1, 1), 2, (257, 512), [10, 3, 2, 4, 8, 1, 7, 1, 2, 1, 2, 1, 1, 7, 2, 8, 0, 2, 0]),
    ("one wave, 560 workgroups", (60, 16, 14, 14, 64, 3, 3, 1, 1), "bf16", (1, 1), 1, (513, 9999), [20, 3, 2, 4, 8, 1, 7, 1, 2, 1, 2, 1, 1, 7, 2, 8, 0, 2, 0]),
    ("two waves, 280 workgroups, 96 accumulators", (280, 16, 13, 13, 64, 3, 3, 1, 1), "bf16", (2, 1), 1, (257, 512), [280, 1, 1, 2, 2, 16, 1, 1, 13, 1, 1, 1, 1, 13, 2, 8, 0, 2, 0]),
    ("three waves", (2, 16, 9, 9, 32, 3, 3, 1, 1), "bf16", (1, 3), 1, (1, 512), [1, 2, 1, 8, 4, 1, 3, 1, 1, 3, 1, 3, 1, 3, 2, 8, 0, 2, 0]),
]


def _defs(op, cfg):
    return dict(t[2:].split("=") for t in P.opevo_kernel_defines(op, P.OPEVO_TILE4L, cfg).split(":", 1)[1].split() if "=" in t)


@pytest.mark.parametrize("label,dims,dtype,waves,shared,grid,cfg", CASES, ids=[c[0] for c in CASES])
def test_plan(label, dims, dtype, waves, shared, grid, cfg):
    op = P.opevo_op_create(P.OPEVO_CONV2D, dims, synth.DTYPE_CODE[dtype])
    plan, D = P.opevo_kernel_plan(op, P.OPEVO_TILE4L, cfg), _defs(op, cfg)
    assert plan.status == P.OPEVO_OK and plan.path == 5 and (int(D["WM"]), int(D["WN"])) == waves
    assert grid[0] <= plan.grid[0] * plan.grid[1] <= grid[1]
    assert int(D["KW"]) == shared and plan.block == 64 * waves[0] * waves[1] * shared
    kernel, _ = P.opevo_kernel_build(op, P.OPEVO_TILE4L, cfg)
    P.opevo_kernel_destroy(kernel)


def test_a_tile_has_no_more_waves_than_steps():
    op = P.opevo_op_create(P.OPEVO_CONV2D, (2, 16, 9, 9, 32, 1, 1, 1, 0), P.OPEVO_BF16)
    cfg = [1, 2, 1, 16, 1, 2, 1, 1, 9, 1, 1, 1, 1, 9, 1, 16, 0, 2, 0]
    assert P.opevo_kernel_plan(op, P.OPEVO_TILE4L, cfg).path == 5 and _defs(op, cfg)["KW"] == "1"


@pytest.mark.gpu
@pytest.mark.parametrize("label,dims,dtype,waves,shared,grid,cfg", CASES, ids=[c[0] for c in CASES])
def test_results_match_the_oracle(label, dims, dtype, waves, shared, grid, cfg):
    """Products of 16-bit values are exact in fp32; sums of at most 800 of them: 1e-5 is 80 roundings."""
    import torch
    from oracle import tensor as T
    x, w = synth.conv_inputs(*dims[:7], dtype, 5)
    want = T.conv2d(x, w, dims[7], dims[8])
    op = P.opevo_op_create(P.OPEVO_CONV2D, dims, synth.DTYPE_CODE[dtype])
    dx, dw = synth.to_device(x, dtype), synth.to_device(w, dtype)
    dy = torch.full((want.size,), float("nan"), device="cuda:0")
    kernel, _ = P.opevo_kernel_build(op, P.OPEVO_TILE4L, cfg)
    for _ in range(3):
        P.opevo_kernel_launch(kernel, dw.data_ptr(), dx.data_ptr(), dy.data_ptr(), torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    P.opevo_kernel_destroy(kernel)
    got = dy.cpu().numpy().astype(np.float64)
    assert np.all(np.isfinite(got)) and np.linalg.norm(got - want.ravel()) <= 1e-5 * np.linalg.norm(want), label
