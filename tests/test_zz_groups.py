"""Direct-to-LDS members whose reduction two groups of waves share: which members do, and their results -- one, two and four
waves per group, slab counts that are no multiple of a group's ring, a transposed first operand, several batches per workgroup,
both atoms, a packed second operand, a reduction split over workgroups on top."""
import numpy as np
import pytest

import paper_2006_05664_amd as P
from paper_2006_05664_amd import synth

V4, V4A, V4K, V4T = P.OPEVO_TILE4, P.OPEVO_TILE4A, P.OPEVO_TILE4K, P.OPEVO_TILE4T
CASES = [   # label, kind, dims, dtype, space, configuration
    ("one wave, 8 slabs of 64", P.OPEVO_MATMUL, (96, 160, 512), "bf16", V4, [3, 1, 1, 32, 5, 1, 1, 32, 8, 64, 1]),
    ("one wave, 5 slabs of 32 per group", P.OPEVO_MATMUL, (64, 96, 320), "f16", V4, [2, 1, 1, 32, 3, 1, 1, 32, 10, 32, 1]),
    ("one wave of 32 x 64, 14 slabs per group in a ring of 3", P.OPEVO_MATMUL, (64, 128, 1792), "bf16", V4, [2, 1, 1, 32, 2, 1, 2, 32, 28, 64, 1]),
    ("two waves, 12 KB slabs", P.OPEVO_MATMUL, (160, 128, 1152), "bf16", V4, [5, 1, 1, 32, 2, 2, 1, 32, 18, 64, 1]),
    ("four waves, slabs of 32", P.OPEVO_MATMUL, (128, 64, 1088), "bf16", V4, [2, 2, 1, 32, 1, 2, 1, 32, 34, 32, 1]),
    ("batches, two per workgroup", P.OPEVO_BMM, (6, 32, 64, 512), "f16", V4, [3, 2, 1, 1, 1, 32, 2, 1, 1, 32, 16, 32, 1]),
    ("first operand transposed", P.OPEVO_BMM_TA, (4, 64, 32, 512), "bf16", V4, [2, 2, 2, 1, 1, 32, 1, 1, 1, 32, 8, 64, 1]),
    ("16x16x32 atoms, slabs of 32", P.OPEVO_MATMUL, (64, 96, 384), "bf16", V4A, [2, 1, 1, 32, 3, 1, 1, 32, 12, 32, 1, 1]),
    ("second operand packed", P.OPEVO_MATMUL, (64, 96, 512), "bf16", V4T, [2, 1, 1, 32, 3, 1, 1, 32, 8, 64, 1, 1]),
    ("reduction split over 2 workgroups as well", P.OPEVO_MATMUL, (64, 96, 1024), "bf16", V4K, [2, 1, 1, 32, 3, 1, 1, 32, 2, 8, 64, 1]),
]


def _defs(op, variant, cfg):
    return dict(t[2:].split("=") for t in P.opevo_kernel_defines(op, variant, cfg).split(":", 1)[1].split() if "=" in t)


@pytest.mark.parametrize("label,kind,dims,dtype,variant,cfg", CASES, ids=[c[0] for c in CASES])
def test_plan(label, kind, dims, dtype, variant, cfg):
    op = P.opevo_op_create(kind, dims, synth.DTYPE_CODE[dtype])
    plan, D = P.opevo_kernel_plan(op, variant, cfg), _defs(op, variant, cfg)
    nw = int(D["WM"]) * int(D["WN"])
    assert plan.status == P.OPEVO_OK and plan.path == 3 and D["KGRP"] == "2" and plan.block == 128 * nw == 2 * int(D["NT"])
    assert int(D["KSTEPS"]) % 2 == 0 and int(D["NSTG"]) % 2 == 0 and int(D["NSTG"]) // 2 >= 2
    stage = (plan.tile[0] + plan.tile[1]) * plan.tile[2] * 2
    assert plan.lds_bytes == int(D["NSTG"]) * stage <= 160 * 1024
    assert nw * plan.wave_tile[0] * plan.wave_tile[1] * 4 <= plan.lds_bytes            # the second group's sum fits the ring
    assert (int(D["NSTG"]) // 2 - 2) * (stage // (1024 * nw)) <= 63                    # the wait count of a group fits its 6 bits
    kernel, _ = P.opevo_kernel_build(op, variant, cfg)
    assert 1000 < P.opevo_kernel_code_size(kernel) < (128 << 10)
    P.opevo_kernel_destroy(kernel)


@pytest.mark.parametrize("dims,cfg", [
    ((96, 160, 448), [3, 1, 1, 32, 5, 1, 1, 32, 7, 64, 1]),            # an odd number of slabs
    ((96, 160, 256), [3, 1, 1, 32, 5, 1, 1, 32, 4, 64, 1]),            # too few
    ((992, 992, 512), [31, 1, 1, 32, 31, 1, 1, 32, 8, 64, 1]),         # several workgroups per compute unit
    ((512, 1024, 1024), [8, 2, 1, 32, 16, 2, 1, 32, 16, 64, 1]),       # bound by what a compute unit can load
    ((512, 1024, 1024), [8, 1, 2, 32, 16, 1, 2, 32, 16, 64, 1]),       # wave tiles of more than two atoms: never measured
    ((512, 1024, 1024), [4, 1, 4, 32, 32, 1, 1, 32, 32, 32, 1]),
    ((256, 256, 256), [1, 1, 2, 128, 8, 1, 1, 32, 8, 32, 1]),
    ((256, 256, 256), [2, 1, 4, 32, 8, 1, 1, 32, 8, 32, 1]),
    ((256, 256, 256), [4, 1, 2, 32, 4, 1, 8, 8, 8, 32, 1]),
    ((256, 256, 256), [8, 1, 32, 1, 2, 1, 16, 8, 8, 32, 1]),
    ((256, 256, 256), [8, 1, 32, 1, 8, 1, 1, 32, 8, 32, 1]),           # reductions of at most 256
])
def test_members_that_keep_one_group(dims, cfg):
    op = P.opevo_op_create(P.OPEVO_MATMUL, dims, P.OPEVO_BF16)
    assert P.opevo_kernel_plan(op, V4, cfg).path == 3 and "KGRP" not in _defs(op, V4, cfg)


@pytest.mark.gpu
@pytest.mark.parametrize("label,kind,dims,dtype,variant,cfg", CASES, ids=[c[0] for c in CASES])
def test_results_match_the_oracle(label, kind, dims, dtype, variant, cfg):
    """Products of 16-bit values are exact in fp32; sums of at most 1792 of them: 1e-5 is 80 roundings."""
    import torch
    from oracle import tensor as T
    make = {P.OPEVO_MATMUL: synth.matmul_inputs, P.OPEVO_BMM: synth.bmm_inputs, P.OPEVO_BMM_TA: synth.bmm_ta_inputs}[kind]
    a, b = make(*dims, dtype, 5)
    want = T.matmul(a, b) if kind == P.OPEVO_MATMUL else T.bmm(a if kind == P.OPEVO_BMM else np.ascontiguousarray(a.transpose(0, 2, 1)), b)
    op = P.opevo_op_create(kind, dims, synth.DTYPE_CODE[dtype])
    da, db = synth.to_device(a, dtype), synth.to_device(b, dtype)
    dc = torch.full((want.size,), float("nan"), device="cuda:0")
    kernel, _ = P.opevo_kernel_build(op, variant, cfg)
    for _ in range(3):
        P.opevo_kernel_launch(kernel, da.data_ptr(), db.data_ptr(), dc.data_ptr(), torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    P.opevo_kernel_destroy(kernel)
    got = dc.cpu().numpy().astype(np.float64)
    assert np.all(np.isfinite(got)) and np.linalg.norm(got - want.ravel()) <= 1e-5 * np.linalg.norm(want), label
