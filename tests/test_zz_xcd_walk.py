"""Workgroups dealt to tiles XCD by XCD: that every tile is dealt once, which members are dealt that way, and their results."""
import ctypes
import re

import numpy as np
import pytest

import paper_2006_05664_amd as P
from host_code import compile_common
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
    """block_id() as the kernels compile it, for every workgroup of a grid in launch order."""
    lib = compile_common("-DOP=1 -DIN_DTYPE=1 -DXCD_WALK=%d -DGRID_N1=%d -DGRID_M1=%d -DGRID_B1=%d" % (walk, n1, m1, b1), """
extern "C" void tiles(int *out)
{
    for (blockIdx.z = 0; blockIdx.z < GRID_B1; ++blockIdx.z)
        for (blockIdx.y = 0; blockIdx.y < GRID_M1; ++blockIdx.y)
            for (blockIdx.x = 0; blockIdx.x < GRID_N1; ++blockIdx.x) { const BlockId id = block_id(); *out++ = id.n; *out++ = id.m; *out++ = id.b; }
}
""")
    total = n1 * m1 * b1
    out = np.full((total, 3), -1, dtype=np.int32)
    lib.tiles(out.ctypes.data_as(ctypes.c_void_p))
    n, m, b = out.T
    assert n.min() >= 0 and m.min() >= 0 and b.min() >= 0 and n.max() < n1 and m.max() < m1 and b.max() < b1
    assert len({tuple(t) for t in out.tolist()}) == total
    j = b * (n1 * m1) + (m * n1 + n if walk == 1 else n * m1 + m)          # the tile's number, columns or rows first
    for x in range(8):                                     # every eighth workgroup: neighbours, in launch order
        assert (np.diff(j[x::8]) == 1).all()


def test_a_row_that_the_compiler_is_not_to_know_is_row_zero():
    lib = compile_common("-DOP=1 -DIN_DTYPE=1 -DXCD_WALK=1 -DROW_UNKNOWN=1 -DGRID_N1=4 -DGRID_M1=1 -DGRID_B1=32",
                         'extern "C" int row(int x, int z) { blockIdx.x = x; blockIdx.y = 0; blockIdx.z = z; return block_id().m; }')
    assert {lib.row(x, z) for x in range(4) for z in range(32)} == {0}


CASES = [   # label, kind, dims, dtype, configuration, walk
    ("batches of 5 tiles, 18 MB of operands", P.OPEVO_BMM_TA, (506, 128, 160, 160), "bf16", [506, 1, 1, 2, 1, 64, 5, 1, 1, 32, 5, 32, 1], 1),
    ("fp32 batches of 4 tiles", P.OPEVO_BMM, (330, 64, 256, 64), "f32", [330, 1, 1, 2, 1, 32, 4, 2, 1, 32, 1, 64, 1], 1),
    ("rows first: few rows, columns of 60 bytes", P.OPEVO_MATMUL, (245, 1530, 1590), "bf16", [35, 1, 1, 7, 51, 2, 1, 15, 30, 53, 1], 2),
    ("columns first: 167 rows of tiles", P.OPEVO_MATMUL, (6680, 330, 400), "f16", [167, 2, 1, 20, 11, 1, 1, 30, 8, 50, 1], 1),
    ("scalar tiles", P.OPEVO_BMM_TA, (42, 96, 128, 96), "f32", [42, 1, 4, 24, 1, 1, 4, 4, 1, 8, 24, 4, 0], 1),
    ("scalar sub-tiles one after another", P.OPEVO_BMM_TA, (60, 210, 250, 216), "f16", [60, 1, 5, 7, 2, 3, 1, 5, 50, 1, 1, 216, 0], 1),
    ("register-staged, 32-row atoms", P.OPEVO_BMM, (215, 64, 128, 128), "bf16", [215, 1, 1, 1, 32, 2, 4, 1, 4, 8, 1, 128, 1], 1),
    ("fragments straight from memory, 16-row atoms", P.OPEVO_BMM, (159, 128, 160, 64), "f16", [159, 1, 2, 1, 2, 32, 10, 1, 16, 1, 2, 32, 0], 1),
    ("the same, one row of tiles, two batches a workgroup", P.OPEVO_BMM, (64, 128, 128, 192), "f16", [32, 2, 1, 2, 4, 16, 4, 1, 2, 16, 1, 192, 0], 1),
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


def test_which_paths_walk_and_where_the_row_is_kept_from_the_compiler():
    walking = [(_walk(kind, dims, dtype, cfg)[0:2], label, cfg) for label, kind, dims, dtype, cfg, walk in CASES if walk]
    assert {plan.path for (_, plan), _, _ in walking} >= {0, 1, 2, 3, 4, 6}
    for (op, plan), label, cfg in walking:
        d = P.opevo_kernel_defines(op, P.OPEVO_TILE4, cfg)
        assert ("ROW_UNKNOWN" in d) == (label == "the same, one row of tiles, two batches a workgroup"), label
        assert ("SUBM" in d) == ("sub-tiles" in label)


def test_a_member_that_spills_walked_is_built_in_the_natural_order_too():
    """One that spills either way: two compilations."""
    op, plan, walk = _walk(P.OPEVO_BMM, (80, 192, 64, 256), "f16", [40, 2, 1, 1, 2, 96, 2, 1, 16, 2, 1, 256, 1])
    assert walk and plan.path == 1
    before = P.opevo_code_cache_stats()
    kernel, _ = P.opevo_kernel_build(op, P.OPEVO_TILE4, [40, 2, 1, 1, 2, 96, 2, 1, 16, 2, 1, 256, 1])
    P.opevo_kernel_destroy(kernel)
    after = P.opevo_code_cache_stats()
    assert after["misses"] - before["misses"] == 2, (before, after)


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
