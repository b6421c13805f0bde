"""The ragged MFMA template keeps the places of a thread's pieces from slab to slab: the offsets it adds to a slab's base, the depth
of its prefetch, and results where slabs, tails and row ends meet."""
import re

import numpy as np
import pytest

import paper_2006_05664_amd as P
from paper_2006_05664_amd import synth

CASES = [   # label, kind, dims, configuration, what the decoder must choose
    ("two slabs on their way, 40 slabs and a tail", P.OPEVO_MATMUL, (120, 90, 1310), [2, 1, 1, 60, 1, 1, 1, 90, 131, 10, 1], dict(DEPTH=2, KEEP=1, NSL=41)),
    ("two on their way, no tail, edges in the last column", P.OPEVO_MATMUL, (100, 95, 2048), [1, 1, 1, 100, 1, 1, 1, 95, 64, 32, 1], dict(DEPTH=2, KEEP=1, NSL=64)),
    ("one on its way, 14 slabs and a tail of two", P.OPEVO_MATMUL, (90, 60, 450), [1, 1, 1, 90, 1, 1, 1, 60, 15, 30, 1], dict(DEPTH=1, KEEP=1, NSL=15)),
    ("one stage, several slabs", P.OPEVO_MATMUL, (45, 50, 300), [1, 1, 1, 45, 1, 2, 1, 25, 5, 60, 0], dict(NSTG=1, KEEP=1)),
    ("transposed first operand, both edges", P.OPEVO_BMM_TA, (3, 27, 35, 330), [3, 1, 3, 1, 1, 9, 5, 1, 1, 7, 6, 55, 1], dict(KEEP=1)),
    ("several batches a workgroup", P.OPEVO_BMM, (6, 25, 40, 250), [2, 3, 1, 1, 1, 25, 1, 1, 1, 40, 5, 50, 1], dict(KEEP=1, BATCH_INNER=3)),
    ("a single slab keeps nothing", P.OPEVO_MATMUL, (27, 35, 20), [3, 1, 1, 9, 5, 1, 1, 7, 1, 20, 1], dict(KEEP=0)),
    ("a tile too large to keep them", P.OPEVO_MATMUL, (231, 945, 330), [7, 1, 11, 3, 1, 9, 21, 5, 330, 1, 1], dict(KEEP=0)),
    ("the same, transposed first operand", P.OPEVO_BMM_TA, (8, 360, 420, 250), [4, 2, 1, 120, 3, 1, 3, 5, 7, 4, 250, 1, 1], dict(KEEP=0)),
]


def _defs(op, cfg):
    return {m.group(1): int(m.group(2)) for m in re.finditer(r"-D(\w+)=(-?\d+)(?:\s|$)", P.opevo_kernel_defines(op, P.OPEVO_TILE4, cfg))}


@pytest.mark.parametrize("label,kind,dims,cfg,want", CASES, ids=[c[0] for c in CASES])
def test_offsets_from_a_slab_s_base(label, kind, dims, cfg, want):
    op = P.opevo_op_create(kind, dims, P.OPEVO_BF16)
    plan, D = P.opevo_kernel_plan(op, P.OPEVO_TILE4, cfg), _defs(op, cfg)
    assert plan.status == P.OPEVO_OK and plan.path == 6 and "KWAVES" not in D and {k: D.get(k) for k in want} == want, D
    KS, NSL, NT, K, N, M, BM, BN = (D[k] for k in "KS NSL NT K N M BM BN".split())
    last0, tail = (NSL - 1) * KS, K % KS != 0
    tail0 = last0 - 8 if NSL > 1 else 0

    def check(pieces, offset, tail_offset, base, tail_base, elements):
        q = np.arange(-(-pieces // NT) * NT)
        q = np.where(q < pieces, q, 0)                      # a thread without a piece loads its operand's first
        for j in range(NSL):
            at = base(j) + offset(q) if not (tail and j == NSL - 1) else tail_base + tail_offset(q)
            assert (offset(q) >= 0).all() and (not tail or (tail_offset(q) >= 0).all()), "an offset is unsigned"
            assert (at >= 0).all() and (at + 8 <= elements).all(), (j, at.min(), at.max())
            yield j, at

    if not D["A_TRANS"]:                                     # pieces along k of BM rows; m0 = the last tile's first row
        ck = KS // 8
        for m0 in {0, M - BM}:
            for j, at in check(BM * ck, lambda q: (q // ck) * K + q % ck * 8, lambda q: (q // ck) * K + np.minimum(last0 + q % ck * 8, K - 8) - tail0,
                               lambda j: m0 * K + j * KS, m0 * K + tail0, M * K):
                assert (at // K == (at + 7) // K).all(), "a piece of a k-contiguous operand stays in its row"
    for width, tile in ((N, BN),) + (((M, BM),) if D["A_TRANS"] else ()):
        c = (tile + 7) // 8
        for x0 in {0, width - tile}:
            place = lambda q: np.minimum(x0 + q % c * 8, width - 8)
            for j, at in check(KS * c, lambda q: (q // c) * width + place(q), lambda q: (np.minimum(last0 + q // c, K - 1) - last0) * width + place(q),
                               lambda j: j * KS * width, last0 * width, K * width):
                assert (at // width == (at + 7) // width).all(), "a piece stays in its row"


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("label,kind,dims,cfg,want", CASES, ids=[c[0] for c in CASES])
def test_results_match_the_oracle(label, kind, dims, cfg, want, dtype):
    """Products of 16-bit values are exact in fp32; sums of at most 2048 of them: 1e-5 is 80 roundings."""
    import torch
    from oracle import tensor as T
    make = {P.OPEVO_MATMUL: synth.matmul_inputs, P.OPEVO_BMM: synth.bmm_inputs, P.OPEVO_BMM_TA: synth.bmm_ta_inputs}[kind]
    a, b = make(*dims, dtype, 5)
    want_c = (T.matmul(a, b) if kind == P.OPEVO_MATMUL else T.bmm(a if kind == P.OPEVO_BMM else np.ascontiguousarray(a.transpose(0, 2, 1)), b)).ravel()
    op = P.opevo_op_create(kind, dims, synth.DTYPE_CODE[dtype])
    da, db = synth.to_device(a, dtype), synth.to_device(b, dtype)
    dc = torch.full((want_c.size,), float("nan"), device="cuda:0")
    kernel, _ = P.opevo_kernel_build(op, P.OPEVO_TILE4, cfg)
    for _ in range(2):
        P.opevo_kernel_launch(kernel, da.data_ptr(), db.data_ptr(), dc.data_ptr(), torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    P.opevo_kernel_destroy(kernel)
    got = dc.cpu().numpy().astype(np.float64)
    assert np.all(np.isfinite(got)) and np.linalg.norm(got - want_c) <= 1e-5 * np.linalg.norm(want_c), label
