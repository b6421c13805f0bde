"""Templates that take a member's workgroup tile alone and divide it by themselves: configurations that differ in nothing else are one program, compiled once."""
import pytest

import paper_2006_05664_amd as P

MM, BMM, CONV = P.OPEVO_MATMUL, P.OPEVO_BMM, P.OPEVO_CONV2D
V, X, L = P.OPEVO_TILE4, P.OPEVO_TILE4X, P.OPEVO_TILE4L
GROUPS = [   # template, kind, dims, dtype, space, configurations of one program, configurations of others
    ("gemm_f32_split", MM, (512, 4096, 1024), P.OPEVO_F32, V,
     [[8, 2, 16, 2, 64, 2, 32, 1, 16, 64, 1], [8, 1, 1, 64, 64, 2, 1, 32, 32, 32, 1], [8, 2, 4, 8, 64, 1, 2, 32, 128, 8, 1]],
     [[16, 1, 1, 32, 64, 2, 1, 32, 16, 64, 1], [8, 2, 16, 2, 128, 1, 1, 32, 16, 64, 1]]),
    ("gemm_f32_split", MM, (128, 64, 928), P.OPEVO_F32, X,
     [[2, 1, 2, 32, 1, 2, 1, 32, 116, 8, 1, 1, 0, 2], [2, 2, 1, 32, 1, 1, 2, 32, 29, 32, 1, 1, 0, 2]], [[2, 1, 2, 32, 1, 2, 1, 32, 116, 8, 1, 1, 0, 0]]),
    ("gemm_ragged", MM, (63, 105, 457), P.OPEVO_BF16, V,
     [[3, 1, 1, 21, 3, 1, 1, 35, 457, 1, 1], [3, 3, 7, 1, 3, 5, 1, 7, 1, 457, 1], [3, 1, 7, 3, 3, 1, 5, 7, 457, 1, 0]], [[3, 1, 1, 21, 5, 1, 1, 21, 457, 1, 1]]),
    ("gemm_ragged", BMM, (6, 25, 40, 550), P.OPEVO_BF16, V,
     [[2, 3, 1, 1, 1, 25, 1, 1, 1, 40, 11, 50, 1], [2, 3, 1, 5, 5, 1, 1, 2, 20, 1, 55, 10, 1]], [[3, 2, 1, 1, 1, 25, 1, 1, 1, 40, 11, 50, 1]]),
    ("conv_strip", CONV, (257, 32, 14, 14, 32, 3, 3, 1, 1), P.OPEVO_BF16, L,
     [[257, 1, 1, 1, 1, 32, 1, 7, 2, 1, 1, 1, 14, 1, 2, 16, 1, 2, 0], [257, 1, 1, 1, 1, 32, 1, 7, 1, 2, 1, 1, 7, 2, 2, 16, 0, 2, 0]],
     [[257, 1, 1, 1, 1, 32, 2, 7, 1, 1, 1, 1, 14, 1, 2, 16, 0, 2, 0]]),
]


@pytest.mark.parametrize("tmpl,kind,dims,dtype,variant,same,others", GROUPS, ids=["%s %d" % (g[0], i) for i, g in enumerate(GROUPS)])
def test_one_program(tmpl, kind, dims, dtype, variant, same, others):
    op = P.opevo_op_create(kind, dims, dtype)
    texts = [P.opevo_kernel_defines(op, variant, cfg) for cfg in same + others]
    assert all(P.opevo_kernel_plan(op, variant, cfg).status == P.OPEVO_OK for cfg in same + others)
    assert all(t.split(":")[0] == tmpl for t in texts[:len(same)]), texts
    assert len(set(texts[:len(same)])) == 1, texts[:len(same)]
    assert len(set(texts)) == 1 + len(others)


def test_it_is_compiled_once(tmp_path):
    _, kind, dims, dtype, variant, same, _ = GROUPS[0]
    op = P.opevo_op_create(kind, dims, dtype)
    P.opevo_code_cache_configure(str(tmp_path), 0)
    try:
        for cfg in same:
            kernel, _ = P.opevo_kernel_build(op, variant, cfg)
            P.opevo_kernel_destroy(kernel)
    finally:
        P.opevo_code_cache_configure(None, 256 << 20)
    assert len(list(tmp_path.iterdir())) == 1
