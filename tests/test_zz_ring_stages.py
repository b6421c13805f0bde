"""Stages of the direct-to-LDS template's ring on grids that do not fit the chip at once: how many a member has, and results with two and three of them."""
import re

import numpy as np
import pytest

import paper_2006_05664_amd as P
from paper_2006_05664_amd import synth

MM, BMM, BMT = P.OPEVO_MATMUL, P.OPEVO_BMM, P.OPEVO_BMM_TA
CASES = [   # label, kind, dims, configuration, stages, waves, bytes of a stage
    ("256 workgroups: one each", BMM, (256, 128, 64, 192), [256, 1, 1, 2, 1, 64, 1, 1, 1, 64, 3, 64, 1], 4, 2, 24576),
    ("600: three fit with two stages, not two", BMM, (600, 128, 64, 192), [600, 1, 1, 2, 1, 64, 1, 1, 1, 64, 3, 64, 1], 2, 2, 24576),
    ("300: two fit with three stages", BMM, (300, 128, 64, 128), [300, 1, 1, 2, 1, 64, 1, 1, 1, 64, 2, 64, 1], 3, 2, 24576),
    ("780: none fits, three stages for two workgroups", BMT, (780, 128, 64, 128), [780, 1, 1, 2, 1, 64, 1, 1, 1, 64, 2, 64, 1], 3, 2, 24576),
    ("three slabs on two stages, four waves", MM, (2304, 2304, 192), [18, 2, 1, 64, 18, 2, 1, 64, 3, 64, 1], 2, 4, 32768),
    ("one wave, none fits, two stages", BMT, (1300, 64, 64, 128), [1300, 1, 1, 1, 1, 64, 1, 1, 1, 64, 2, 64, 1], 2, 1, 16384),
    ("three waves on a compute unit, none fits: as it was", BMT, (1600, 64, 32, 128), [1600, 1, 1, 1, 1, 64, 1, 1, 1, 32, 2, 64, 1], 4, 1, 12288),
    ("three waves on a compute unit, four fit", BMM, (800, 64, 32, 128), [800, 1, 1, 1, 1, 64, 1, 1, 1, 32, 2, 64, 1], 3, 1, 12288),
    ("twelve waves: as it was", MM, (2816, 2240, 96), [44, 2, 1, 32, 70, 1, 1, 32, 3, 32, 1], 4, 2, 6144),
]

@pytest.mark.parametrize("label,kind,dims,cfg,stages,waves,stage", CASES, ids=[c[0] for c in CASES])
def test_stages(label, kind, dims, cfg, stages, waves, stage):
    op = P.opevo_op_create(kind, dims, P.OPEVO_BF16)
    plan = P.opevo_kernel_plan(op, P.OPEVO_TILE4, cfg)
    assert plan.status == P.OPEVO_OK and plan.path == 3, plan.reason
    D = {k: int(v) for k, v in re.findall(r"-D(\w+)=(-?\d+)(?=\s|$)", P.opevo_kernel_defines(op, P.OPEVO_TILE4, cfg))}
    assert plan.block == 64 * waves and (D["BM"] + D["BN"]) * D["BK"] * 2 == stage and plan.lds_bytes == stages * stage
    assert (D["NSTG"], D["NSTAGE"]) == (stages, stages) and "KGRP" not in D


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("label,kind,dims,cfg,stages,waves,stage", CASES, ids=[c[0] for c in CASES])
def test_results_match_the_reference(label, kind, dims, cfg, stages, waves, stage, dtype):
    """Products of 16-bit values are exact in fp32; sums of at most 192 of them: 1e-5 is 80 roundings."""
    import torch
    op = P.opevo_op_create(kind, dims, synth.DTYPE_CODE[dtype])
    a, b = {MM: synth.matmul_inputs, BMM: synth.bmm_inputs, BMT: synth.bmm_ta_inputs}[kind](*dims, dtype, 3)
    da, db = synth.to_device(a, dtype), synth.to_device(b, dtype)
    x, y = da.double(), db.double()
    want = torch.matmul(x.transpose(-1, -2).contiguous() if kind == BMT else x, y).ravel()
    dc = torch.full((want.numel(),), float("nan"), device="cuda:0")
    kernel, _ = P.opevo_kernel_build(op, P.OPEVO_TILE4, cfg)
    for _ in range(2):                                     # the second launch overwrites what the first one left
        P.opevo_kernel_launch(kernel, da.data_ptr(), db.data_ptr(), dc.data_ptr(), torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    P.opevo_kernel_destroy(kernel)
    got = dc.double()
    assert bool(torch.isfinite(got).all()) and float((got - want).norm()) <= 1e-5 * float(want.norm()), label
