"""fp32 members whose output is stored past the L2: which they are, and their results."""
import numpy as np
import pytest

import paper_2006_05664_amd as P
from paper_2006_05664_amd import synth

V, X, K3 = P.OPEVO_TILE4, P.OPEVO_TILE4X, P.OPEVO_TILE4K
CASES = [   # label, kind, dims, variant, configuration, stored past the L2
    ("2 MiB", P.OPEVO_MATMUL, (512, 1024, 64), V, [8, 1, 2, 32, 16, 2, 1, 32, 2, 32, 1], True),
    ("below 2 MiB", P.OPEVO_MATMUL, (480, 1024, 64), V, [15, 1, 1, 32, 16, 2, 1, 32, 2, 32, 1], False),
    ("32 MiB, batches, one stage", P.OPEVO_BMM, (128, 256, 256, 32), V, [128, 1, 4, 2, 1, 32, 4, 1, 2, 32, 2, 16, 1], True),
    ("above 32 MiB", P.OPEVO_BMM, (129, 256, 256, 32), V, [129, 1, 4, 2, 1, 32, 4, 1, 2, 32, 2, 16, 1], False),
    ("transposed first operand, K = 224", P.OPEVO_BMM_TA, (40, 96, 160, 224), V, [40, 1, 1, 3, 1, 32, 5, 1, 1, 32, 14, 16, 1], True),
    ("K = 256", P.OPEVO_BMM_TA, (40, 96, 160, 256), V, [40, 1, 1, 3, 1, 32, 5, 1, 1, 32, 16, 16, 1], False),
    ("tiles computed one after another, one wave of two", P.OPEVO_MATMUL, (2048, 512, 96), V, [2, 32, 1, 32, 16, 1, 1, 32, 3, 32, 0], True),
    ("a launch order of its own", P.OPEVO_MATMUL, (512, 1024, 64), X, [8, 1, 2, 32, 16, 2, 1, 32, 2, 32, 1, 1, 0, 2], True),
    ("split reduction", P.OPEVO_MATMUL, (512, 1024, 64), K3, [8, 1, 2, 32, 16, 2, 1, 32, 2, 1, 32, 1], False),
]


def _member(kind, dims, variant, cfg):
    op = P.opevo_op_create(kind, dims, P.OPEVO_F32)
    plan = P.opevo_kernel_plan(op, variant, cfg)
    assert plan.status == P.OPEVO_OK and plan.path == 4
    return op, "-DNT_OUT=1" in P.opevo_kernel_defines(op, variant, cfg)


@pytest.mark.parametrize("label,kind,dims,variant,cfg,past", CASES, ids=[c[0] for c in CASES])
def test_which_outputs_go_past_the_l2(label, kind, dims, variant, cfg, past):
    assert _member(kind, dims, variant, cfg)[1] == past


@pytest.mark.gpu
@pytest.mark.parametrize("label,kind,dims,variant,cfg,past", [c for c in CASES if c[-1]], ids=[c[0] for c in CASES if c[-1]])
def test_results_match_the_oracle(label, kind, dims, variant, cfg, past):
    """Sums of at most 224 rounded products in fp32: 1e-5 is 80 roundings."""
    import torch
    from oracle import tensor as T
    make = {P.OPEVO_MATMUL: synth.matmul_inputs, P.OPEVO_BMM: synth.bmm_inputs, P.OPEVO_BMM_TA: synth.bmm_ta_inputs}[kind]
    a, b = make(*dims, "f32", 5)
    want = (T.matmul(a, b) if kind == P.OPEVO_MATMUL else T.bmm(a if kind == P.OPEVO_BMM else np.ascontiguousarray(a.transpose(0, 2, 1)), b)).ravel()
    op, _ = _member(kind, dims, variant, cfg)
    da, db = synth.to_device(a, "f32"), synth.to_device(b, "f32")
    dc = torch.full((want.size,), float("nan"), device="cuda:0")
    kernel, _ = P.opevo_kernel_build(op, variant, cfg)
    for _ in range(2):                                     # the second launch overwrites what the first one left
        P.opevo_kernel_launch(kernel, da.data_ptr(), db.data_ptr(), dc.data_ptr(), torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    P.opevo_kernel_destroy(kernel)
    got = dc.cpu().numpy().astype(np.float64)
    assert np.all(np.isfinite(got)) and np.linalg.norm(got - want) <= 1e-5 * np.linalg.norm(want), label
