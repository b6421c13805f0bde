"""Conv2d members that ask for the two-stage loop on an image patch, on more workgroups than compute units: the row-strip template runs them."""
import numpy as np
import pytest

import paper_2006_05664_amd as P
from paper_2006_05664_amd import synth

V = P.OPEVO_TILE4L
CASES = [   # label, dims, configuration, template
    ("257 workgroups", (257, 32, 14, 14, 32, 3, 3, 1, 1), [257, 1, 1, 1, 1, 32, 1, 7, 2, 1, 1, 1, 14, 1, 2, 16, 1, 2, 0], "conv_strip"),
    ("256 workgroups", (256, 32, 14, 14, 32, 3, 3, 1, 1), [256, 1, 1, 1, 1, 32, 1, 7, 2, 1, 1, 1, 14, 1, 2, 16, 1, 2, 0], "conv_patch"),
    ("odd width, 5x5", (10, 64, 27, 27, 96, 5, 5, 1, 2), [10, 1, 3, 1, 1, 32, 9, 3, 1, 1, 1, 1, 27, 1, 4, 16, 1, 2, 0], "conv_strip"),
    ("one tap, four slabs", (50, 64, 28, 28, 32, 1, 1, 1, 0), [50, 1, 1, 1, 1, 32, 7, 4, 1, 1, 1, 1, 28, 1, 4, 16, 1, 2, 0], "conv_strip"),
    ("two pixel waves", (300, 32, 14, 14, 32, 3, 3, 1, 1), [300, 1, 1, 1, 1, 32, 1, 2, 7, 1, 1, 1, 14, 1, 2, 16, 1, 2, 0], "conv_patch"),
    ("waves that share a tile", (257, 32, 14, 14, 32, 3, 3, 1, 1), [257, 1, 1, 1, 1, 32, 1, 7, 2, 1, 1, 1, 14, 1, 2, 16, 1, 2, 1], "conv_patch"),
]


@pytest.mark.parametrize("label,dims,cfg,tmpl", CASES, ids=[c[0] for c in CASES])
def test_template(label, dims, cfg, tmpl):
    op = P.opevo_op_create(P.OPEVO_CONV2D, dims, P.OPEVO_BF16)
    plan = P.opevo_kernel_plan(op, V, cfg)
    assert plan.status == P.OPEVO_OK and plan.path == 5, plan.reason
    assert P.opevo_kernel_defines(op, V, cfg).split(":")[0] == tmpl


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("label,dims,cfg,tmpl", CASES, ids=[c[0] for c in CASES])
def test_results_match_the_oracle(label, dims, cfg, tmpl, dtype):
    """Products of 16-bit values are exact in fp32; sums of at most 1600 of them, in any order: 1e-5 is 80 roundings."""
    import torch
    from oracle import tensor as T
    img, ker = synth.conv_inputs(*dims[:7], dtype, 9)
    want = T.conv2d(img, ker, dims[7], dims[8]).ravel()
    op = P.opevo_op_create(P.OPEVO_CONV2D, dims, synth.DTYPE_CODE[dtype])
    dk, di = synth.to_device(ker, dtype), synth.to_device(img, dtype)
    dc = torch.full((want.size,), float("nan"), device="cuda:0")
    kernel, _ = P.opevo_kernel_build(op, V, cfg)
    for _ in range(2):                                     # the second launch overwrites what the first one left
        P.opevo_kernel_launch(kernel, dk.data_ptr(), di.data_ptr(), dc.data_ptr(), torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    P.opevo_kernel_destroy(kernel)
    got = dc.cpu().numpy().astype(np.float64)
    assert np.all(np.isfinite(got)) and np.linalg.norm(got - want) <= 1e-5 * np.linalg.norm(want), label
