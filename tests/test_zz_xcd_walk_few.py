"""Grids that do not fill the chip, where an XCD has an eighth of the tiles and no more: which of them are dealt XCD by XCD, and their results on every template."""
import re

import numpy as np
import pytest

import paper_2006_05664_amd as P
from paper_2006_05664_amd import synth

CASES = [   # label, dims, dtype, configuration, template, walk
    ("66 tiles", (2112, 128, 1088), "bf16", [33, 2, 1, 32, 2, 2, 1, 32, 17, 64, 1], "gemm_mfma_dlds", 1),
    ("one row of 109 tiles, the shortest reduction", (64, 3488, 1056), "f16", [1, 2, 1, 32, 109, 1, 1, 32, 33, 32, 1], "gemm_mfma_dlds", 1),
    ("a shorter reduction", (64, 3488, 1024), "f16", [1, 2, 1, 32, 109, 1, 1, 32, 32, 32, 1], "gemm_mfma_dlds", 0),
    ("register-staged, 16-row atoms", (1056, 64, 2048), "bf16", [66, 1, 1, 16, 2, 2, 1, 16, 64, 32, 0], "gemm_mfma", 1),
    ("odd extents", (60, 3360, 1367), "f16", [2, 1, 1, 30, 105, 1, 1, 32, 1367, 1, 1], "gemm_ragged", 2),
    ("fp32", (96, 4224, 544), "f32", [3, 1, 1, 32, 66, 2, 1, 32, 17, 32, 1], "gemm_f32_split", 2),
    ("scalar tiles", (96, 928, 3008), "f32", [2, 3, 4, 4, 116, 2, 4, 1, 188, 16, 0], "gemm_scalar", 0),
]


def _member(dims, dtype, cfg):
    op = P.opevo_op_create(P.OPEVO_MATMUL, dims, synth.DTYPE_CODE[dtype])
    text = P.opevo_kernel_defines(op, P.OPEVO_TILE4, cfg)
    walk = re.search(r"-DXCD_WALK=(\d)", text)
    return op, text.split(":")[0], int(walk.group(1)) if walk else 0


@pytest.mark.parametrize("label,dims,dtype,cfg,template,walk", CASES, ids=[c[0] for c in CASES])
def test_which_of_them_are_dealt_by_xcd(label, dims, dtype, cfg, template, walk):
    assert _member(dims, dtype, cfg)[1:] == (template, walk)


@pytest.mark.gpu
@pytest.mark.parametrize("label,dims,dtype,cfg,template,walk", [c for c in CASES if c[-1]], ids=[c[0] for c in CASES if c[-1]])
def test_results_match_the_oracle(label, dims, dtype, cfg, template, walk):
    """Sums of at most 2048 products in fp32: 1e-5 is 80 roundings."""
    import torch
    from oracle import tensor as T
    a, b = synth.matmul_inputs(*dims, dtype, 5)
    want = T.matmul(a, b).ravel()
    op = _member(dims, dtype, cfg)[0]
    da, db = synth.to_device(a, dtype), synth.to_device(b, dtype)
    dc = torch.full((want.size,), float("nan"), device="cuda:0")
    kernel, _ = P.opevo_kernel_build(op, P.OPEVO_TILE4, cfg)
    P.opevo_kernel_launch(kernel, da.data_ptr(), db.data_ptr(), dc.data_ptr(), torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    P.opevo_kernel_destroy(kernel)
    got = dc.cpu().numpy().astype(np.float64)
    assert np.all(np.isfinite(got)) and np.linalg.norm(got - want) <= 1e-5 * np.linalg.norm(want), label
