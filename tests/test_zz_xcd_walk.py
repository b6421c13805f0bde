"""Workgroups dealt to tiles XCD by XCD: that every tile is dealt once, which members are dealt that way, and their results."""
import re

import numpy as np
import pytest

import paper_2006_05664_amd as P
from paper_2006_05664_amd import synth


def _walk(kind, dims, dtype, cfg, variant=P.OPEVO_TILE4):
    op = P.opevo_op_create(kind, dims, synth.DTYPE_CODE[dtype])
    plan = P.opevo_kernel_plan(op, variant, cfg)
    d = {m.group(1): int(m.group(2)) for m in re.finditer(r"-D(\w+)=(-?\d+)(?:\s|$)", P.opevo_kernel_defines(op, variant, cfg))}
    assert plan.status == P.OPEVO_OK and ("XCD_WALK" not in d or [d["GRID_N1"], d["GRID_M1"], d["GRID_B1"]] == list(plan.grid))
    return op, plan, d.get("XCD_WALK", 0)


@pytest.mark.parametrize("n1,m1,b1", [(1, 1, 1), (3, 1, 2), (7, 5, 1), (8, 8, 1), (55, 167, 1), (13, 1, 9), (5, 3, 31), (1, 64, 1), (64, 1, 1), (9, 11, 13)])
@pytest.mark.parametrize("walk", [1, 2])
def test_every_tile_is_dealt_once_and_an_xcd_walks_neighbours(n1, m1, b1, walk):
    total = n1 * m1 * b1
    L = np.arange(total)
    xcd = L % 8
    j = xcd * (total // 8) + np.minimum(xcd, total % 8) + L // 8
    assert np.array_equal(np.sort(j), L)
    for x in range(8):                                     # contiguous, in launch order
        assert (np.diff(j[xcd == x]) == 1).all()
    inside = j % (n1 * m1)
    n, m, b = (inside % n1, inside // n1, j // (n1 * m1)) if walk == 1 else (inside // m1, inside % m1, j // (n1 * m1))
    assert len(set(zip(n.tolist(), m.tolist(), b.tolist()))) == total and n.max() < n1 and m.max() < m1 and b.max() < b1


CASES = [   # label, kind, dims, dtype, configuration, walk
    ("batches of 5 tiles, 18 MB of operands", P.OPEVO_BMM_TA, (506, 128, 160, 160), "bf16", [506, 1, 1, 2, 1, 64, 5, 1, 1, 32, 5, 32, 1], 1),
    ("fp32 batches of 4 tiles", P.OPEVO_BMM, (330, 64, 256, 64), "f32", [330, 1, 1, 2, 1, 32, 4, 2, 1, 32, 1, 64, 1], 1),
    ("rows first: few rows, columns of 60 bytes", P.OPEVO_MATMUL, (245, 1530, 1590), "bf16", [35, 1, 1, 7, 51, 2, 1, 15, 30, 53, 1], 2),
    ("columns first: 167 rows of tiles", P.OPEVO_MATMUL, (6680, 330, 400), "f16", [167, 2, 1, 20, 11, 1, 1, 30, 8, 50, 1], 1),
    ("operands that an L2 holds", P.OPEVO_MATMUL, (1000, 1000, 1000), "bf16", [50, 4, 1, 5, 10, 5, 20, 1, 10, 100, 1], 0),
    ("a grid whose natural order gives an XCD a square", P.OPEVO_MATMUL, (8192, 8192, 8192), "bf16", [32, 2, 2, 64, 32, 4, 2, 32, 128, 64, 1], 0),
    ("small batches", P.OPEVO_BMM, (52, 224, 192, 64), "bf16", [52, 1, 7, 1, 1, 32, 3, 2, 1, 32, 1, 64, 1], 0),
]


@pytest.mark.parametrize("label,kind,dims,dtype,cfg,walk", CASES, ids=[c[0] for c in CASES])
def test_which_members_are_dealt_by_xcd(label, kind, dims, dtype, cfg, walk):
    assert _walk(kind, dims, dtype, cfg)[2] == walk


def test_split_reductions_and_chosen_launch_orders_keep_their_own():
    assert _walk(P.OPEVO_MATMUL, (2496, 7072, 6848), "bf16", [39, 1, 2, 32, 221, 1, 1, 32, 2, 107, 32, 1], P.OPEVO_TILE4K)[2] == 0
    assert _walk(P.OPEVO_MATMUL, (2496, 7072, 6848), "bf16", [39, 1, 2, 32, 221, 1, 1, 32, 214, 32, 1, 0, 1, 0], P.OPEVO_TILE4X)[2] == 0


@pytest.mark.gpu
@pytest.mark.parametrize("label,kind,dims,dtype,cfg,walk", [c for c in CASES if c[-1]], ids=[c[0] for c in CASES if c[-1]])
def test_results_match_the_oracle(label, kind, dims, dtype, cfg, walk):
    """Sums of at most 1590 products in fp32: 1e-5 is 80 roundings (fp32 inputs: products are rounded too)."""
    import torch
    from oracle import tensor as T
    make = {P.OPEVO_MATMUL: synth.matmul_inputs, P.OPEVO_BMM: synth.bmm_inputs, P.OPEVO_BMM_TA: synth.bmm_ta_inputs}[kind]
    a, b = make(*dims, dtype, 5)
    want = (T.matmul(a, b) if kind == P.OPEVO_MATMUL else T.bmm(a if kind == P.OPEVO_BMM else np.ascontiguousarray(a.transpose(0, 2, 1)), b)).ravel()
    op, _, _ = _walk(kind, dims, dtype, cfg)
    da, db = synth.to_device(a, dtype), synth.to_device(b, dtype)
    dc = torch.full((want.size,), float("nan"), device="cuda:0")
    kernel, _ = P.opevo_kernel_build(op, P.OPEVO_TILE4, cfg)
    P.opevo_kernel_launch(kernel, da.data_ptr(), db.data_ptr(), dc.data_ptr(), torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    P.opevo_kernel_destroy(kernel)
    got = dc.cpu().numpy().astype(np.float64)
    assert np.all(np.isfinite(got)) and np.linalg.norm(got - want) <= 1e-5 * np.linalg.norm(want), label
