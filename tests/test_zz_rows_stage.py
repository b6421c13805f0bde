"""The few-channels convolution template's kernel tensor, which comes through the LDS: which members have room for it, the words and shifts that a lane's fragment is
made of (re-computed on the CPU), and results for odd and even rows, both atoms, one and two groups of taps, rows of the patch shorter and longer than the tensor's."""
import re

import numpy as np
import pytest

import paper_2006_05664_amd as P
from paper_2006_05664_amd import synth

V4, V4C = P.OPEVO_TILE4, P.OPEVO_TILE4C
CASES = [   # label, dims, space, configuration, 1 = where the patch will be, 2 = beside it, 0 = straight from memory
    ("11 taps, 33 rows of them", (2, 3, 40, 40, 64, 11, 11, 2, 5), V4C, [2, 1, 1, 4, 1, 16, 5, 2, 2, 1, 1, 1, 20, 1, 1, 33, 11, 0, 0], 2),
    ("even rows", (1, 2, 20, 24, 32, 4, 4, 1, 1), V4, [1, 1, 1, 2, 1, 16, 19, 1, 1, 1, 1, 1, 23, 1, 4, 8, 0], 2),
    ("odd rows of an even number of taps", (2, 3, 16, 21, 32, 3, 5, 1, 2), V4, [2, 1, 2, 1, 1, 16, 3, 1, 1, 6, 3, 1, 1, 7, 3, 15, 1], 1),
    ("16-row atoms, three kernel rows of four a step", (1, 5, 17, 18, 48, 7, 7, 2, 3), V4, [1, 1, 1, 3, 1, 16, 9, 1, 1, 1, 1, 1, 9, 1, 5, 49, 0], 2),
    ("16-row atoms, 16 taps", (1, 1, 20, 40, 16, 2, 16, 1, 0), V4, [1, 1, 1, 1, 1, 16, 19, 1, 1, 1, 5, 1, 5, 1, 1, 32, 0], 2),
    ("one tap", (2, 3, 12, 20, 32, 1, 1, 1, 0), V4, [2, 1, 1, 1, 1, 32, 6, 2, 1, 1, 1, 1, 20, 1, 3, 1, 0], 1),
    ("several row blocks, the last ends the tensor", (1, 1, 14, 14, 96, 5, 5, 1, 0), V4, [1, 1, 6, 1, 1, 16, 5, 1, 2, 1, 1, 1, 10, 1, 1, 25, 1], 1),
    ("no room: 12 channels of 7 x 7, 192 rows", (1, 12, 14, 14, 192, 7, 7, 1, 0), V4C, [1, 1, 1, 12, 1, 16, 1, 1, 8, 1, 1, 1, 8, 1, 1, 84, 7, 0, 0], None),
]


def _defs(op, variant, cfg):
    text = P.opevo_kernel_defines(op, variant, cfg)
    return text.split(":")[0], {m.group(1): int(m.group(2)) for m in re.finditer(r"-D(\w+)=(-?\d+)(?=\s|$)", text)}


@pytest.mark.parametrize("label,dims,variant,cfg,stage", CASES, ids=[c[0] for c in CASES])
def test_a_fragment_s_words_and_shift(label, dims, variant, cfg, stage):
    op = P.opevo_op_create(P.OPEVO_CONV2D, dims, P.OPEVO_BF16)
    plan = P.opevo_kernel_plan(op, variant, cfg)
    tmpl, D = _defs(op, variant, cfg)
    if stage is None:
        assert tmpl != "conv_rows" or D["STAGE_A"] == 0
        return
    assert plan.status == P.OPEVO_OK and tmpl == "conv_rows" and D["STAGE_A"] == stage, (plan.reason, tmpl, D.get("STAGE_A"))
    _, CIN, _, _, M, HK, WK, _, _ = dims
    BM, K, atom, NT = D["BM"], CIN * HK * WK, D["ATOM"], D["NT"]
    room = BM * K + 128
    assert BM * K % 8 == 0 and room * 2 <= plan.lds_bytes and room * 2 <= 65536 + 64 * 1024 * (stage == 1)
    assert plan.lds_bytes == D["LDS_BYTES"] <= 160 * 1024 // max(1, 8 // (D["WM"] * D["WN"]))
    Q = D["WKP"] // 8
    RPS = (2 if atom == 32 else 4) // Q
    SPC = -(-HK // RPS)
    rows = np.concatenate([np.arange(BM * K), np.full(128, -1)]).astype(np.int64)          # an element's own number; -1 behind the tensor's
    for row in range(BM):
        for kg in range(2 if atom == 32 else 4):
            first = row * K + kg // Q * WK + kg % Q * 8
            odd, at = first & 1, first >> 1
            for t in range(CIN * SPC):
                step = (t // SPC * HK + t % SPC * RPS) * WK
                w = (at + odd if step & 1 else at) + (step >> 1)
                assert 2 * w + 10 <= room
                words = rows[2 * w:2 * w + 10]
                if K % 2 or WK % 2:
                    words = words[odd ^ (step & 1):]
                else:
                    assert not odd and not step & 1
                for e in range(8):
                    tap, r = kg % Q * 8 + e, t % SPC * RPS + kg // Q
                    if tap < WK and r < HK:                                   # the others are cleared
                        assert words[e] == row * K + (t // SPC * HK + r) * WK + tap


@pytest.mark.gpu
@pytest.mark.parametrize("label,dims,variant,cfg,stage", CASES, ids=[c[0] for c in CASES])
def test_the_plan_counts_all_the_lds(label, dims, variant, cfg, stage):
    """The kernel tensor's rows beside the patch are an array of the kernel's own, which the plan's figure includes."""
    op = P.opevo_op_create(P.OPEVO_CONV2D, dims, P.OPEVO_BF16)
    kernel, _ = P.opevo_kernel_build(op, variant, cfg)
    static = P.opevo_kernel_resources(kernel)["static_lds"]
    P.opevo_kernel_destroy(kernel)
    plan = P.opevo_kernel_plan(op, variant, cfg)
    tmpl, D = _defs(op, variant, cfg)
    assert static == ((D["BM"] * D["K"] + 128) * 2 if tmpl == "conv_rows" and stage == 2 else 0)
    assert static == 0 or static < plan.lds_bytes == D["LDS_BYTES"]


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("label,dims,variant,cfg,stage", CASES[:-1], ids=[c[0] for c in CASES[:-1]])
def test_results_match_the_oracle(label, dims, variant, cfg, stage, dtype):
    """Products of 16-bit values are exact in fp32; sums of at most 363 of them: 1e-5 is 80 roundings.  The values past the tensor's rows are NaN and infinite: none of
    them may reach a sum."""
    import torch
    from oracle import tensor as T
    img, ker = synth.conv_inputs(*dims[:7], dtype, 5)
    want = T.conv2d(img, ker, dims[7], dims[8]).ravel()
    op = P.opevo_op_create(P.OPEVO_CONV2D, dims, synth.DTYPE_CODE[dtype])
    dk, di = synth.to_device(ker, dtype).ravel(), synth.to_device(img, dtype)
    beside = torch.cat([dk, torch.full((64,), float("nan"), device="cuda:0").to(dk.dtype), torch.full((64,), float("inf"), device="cuda:0").to(dk.dtype)])
    dc = torch.full((want.size,), float("nan"), device="cuda:0")
    kernel, _ = P.opevo_kernel_build(op, variant, cfg)
    for _ in range(2):                                     # the second launch overwrites what the first one left
        P.opevo_kernel_launch(kernel, beside.data_ptr(), di.data_ptr(), dc.data_ptr(), torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    P.opevo_kernel_destroy(kernel)
    got = dc.cpu().numpy().astype(np.float64)
    assert np.all(np.isfinite(got)) and np.linalg.norm(got - want) <= 1e-5 * np.linalg.norm(want), label


def test_a_member_that_spills_with_it_keeps_its_template(tmp_path):
    """Straight from memory it does not spill: two compilations, both of this template."""
    op = P.opevo_op_create(P.OPEVO_CONV2D, (33, 3, 224, 224, 128, 11, 11, 4, 0), P.OPEVO_F16)
    cfg = [11, 3, 4, 2, 1, 16, 3, 3, 6, 1, 6, 1, 9, 1, 1, 33, 11, 0, 0]
    assert _defs(op, V4C, cfg)[1]["STAGE_A"] == 1
    P.opevo_code_cache_configure(str(tmp_path), 0)
    try:
        kernel, _ = P.opevo_kernel_build(op, V4C, cfg)
        P.opevo_kernel_destroy(kernel)
    finally:
        P.opevo_code_cache_configure(None, 256 << 20)
    keys = [f.read_bytes().split(b"\x7fELF")[0] for f in tmp_path.iterdir()]
    assert sorted(b"STAGE_A=0" in k for k in keys) == [False, True] and all(b"conv_rows" in k for k in keys)
