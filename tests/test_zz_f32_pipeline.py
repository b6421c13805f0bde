"""The pipelined slab loop of the fp32 MFMA template where its parts meet: slabs of a single group of 8 steps, of an odd number of
groups, two slabs, threads without a piece, a transposed first operand, batches, convolutions with padded slabs and ragged
tiles, folded members.  fp32 sums of at most 768 products: 2e-6 is 16 roundings of the result's norm."""
import numpy as np
import pytest

import paper_2006_05664_amd as P
from paper_2006_05664_amd import synth

pytestmark = pytest.mark.gpu

MM, BMM, TA, CONV = P.OPEVO_MATMUL, P.OPEVO_BMM, P.OPEVO_BMM_TA, P.OPEVO_CONV2D
CASES = [
    ("slabs of one group", MM, (64, 96, 64), [2, 1, 1, 32, 3, 1, 1, 32, 8, 8, 1]),
    ("slabs of three groups", MM, (64, 96, 240), [1, 2, 1, 32, 3, 1, 1, 32, 10, 24, 1]),
    ("two slabs, 64 x 64 wave tiles", MM, (128, 128, 128), [1, 2, 2, 32, 2, 1, 2, 32, 2, 64, 1]),
    ("threads without a piece", MM, (128, 96, 96), [1, 4, 1, 32, 1, 3, 1, 32, 12, 8, 1]),
    ("16 waves", MM, (128, 256, 192), [1, 4, 1, 32, 2, 4, 1, 32, 6, 32, 1]),
    ("batches, two per workgroup", BMM, (6, 64, 32, 96), [3, 2, 2, 1, 1, 32, 1, 1, 1, 32, 12, 8, 1]),
    ("first operand transposed", TA, (4, 64, 96, 160), [2, 2, 1, 2, 1, 32, 3, 1, 1, 32, 10, 16, 1]),
    ("folded: two passes of 16 waves", MM, (256, 256, 128), [1, 8, 1, 32, 2, 4, 1, 32, 8, 16, 1]),
    ("convolution, slabs of 18 padded to 24, ragged tiles", CONV, (2, 16, 9, 9, 64, 3, 3, 1, 1), [1, 2, 2, 1, 1, 32, 3, 1, 1, 3, 3, 1, 1, 3, 8, 18, 1]),
]


@pytest.mark.parametrize("label,kind,dims,cfg", CASES, ids=[c[0] for c in CASES])
def test_results_match_the_oracle(label, kind, dims, cfg):
    import torch
    from oracle import tensor as T
    if kind == CONV:
        img, ker = synth.conv_inputs(*dims[:7], "f32", 5)
        a, b, want = ker, img, T.conv2d(img, ker, dims[7], dims[8])
    else:
        a, b = {MM: synth.matmul_inputs, BMM: synth.bmm_inputs, TA: synth.bmm_ta_inputs}[kind](*dims, "f32", 5)
        want = T.matmul(a, b) if kind == MM else T.bmm(a if kind == BMM else np.ascontiguousarray(a.transpose(0, 2, 1)), b)
    op = P.opevo_op_create(kind, dims, P.OPEVO_F32)
    plan = P.opevo_kernel_plan(op, P.OPEVO_TILE4, cfg)
    assert plan.status == P.OPEVO_OK and plan.path == 4, (plan.path, plan.reason)
    da, db = synth.to_device(a, "f32"), synth.to_device(b, "f32")
    dc = torch.full((want.size,), float("nan"), device="cuda:0")
    kernel, _ = P.opevo_kernel_build(op, P.OPEVO_TILE4, cfg)
    for _ in range(2):
        P.opevo_kernel_launch(kernel, da.data_ptr(), db.data_ptr(), dc.data_ptr(), torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    P.opevo_kernel_destroy(kernel)
    got = dc.cpu().numpy().astype(np.float64)
    assert np.all(np.isfinite(got)) and np.linalg.norm(got - want.ravel()) <= 2e-6 * np.linalg.norm(want), label
