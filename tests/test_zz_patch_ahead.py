"""The convolution template that keeps a patch in the LDS, with two slabs of global loads in flight: which members have them, which slab a pass multiplies (the order of
loads and stores re-computed on the CPU), and results for odd and even numbers of slabs, one tap and nine, odd widths, strides and shared tiles."""
import re

import numpy as np
import pytest

import paper_2006_05664_amd as P
from paper_2006_05664_amd import synth

V = P.OPEVO_TILE4L
CASES = [   # label, dims, configuration, slabs, waves that share a tile, two slabs ahead
    ("one tap, three slabs, odd width", (2, 48, 9, 9, 32, 1, 1, 1, 0), [1, 2, 1, 1, 32, 1, 1, 1, 3, 3, 1, 9, 1, 1, 24, 2, 1, 2, 0], 3, 1, True),
    ("one tap, four slabs", (2, 64, 8, 8, 32, 1, 1, 1, 0), [1, 2, 1, 1, 8, 4, 1, 1, 2, 4, 2, 4, 1, 1, 32, 2, 1, 2, 3], 4, 1, True),
    ("one tap, five slabs, stride 2", (1, 80, 7, 9, 64, 1, 1, 2, 0), [1, 1, 1, 64, 1, 1, 1, 1, 2, 2, 1, 1, 5, 1, 40, 2, 1, 2, 3], 5, 1, True),
    ("one tap, 240 workgroups", (9, 48, 40, 40, 64, 1, 1, 1, 0), [3, 3, 2, 4, 1, 8, 20, 1, 2, 1, 2, 1, 5, 4, 12, 4, 1, 2, 1], 3, 1, True),
    ("nine taps, eight waves", (2, 48, 7, 7, 32, 3, 3, 1, 1), [2, 1, 1, 1, 1, 32, 1, 1, 1, 7, 1, 7, 1, 1, 12, 4, 1, 2, 3], 3, 8, True),
    ("nine taps, two waves, stride 2", (1, 64, 9, 9, 32, 3, 3, 2, 1), [1, 1, 1, 2, 1, 16, 1, 1, 1, 5, 1, 1, 1, 5, 4, 16, 1, 2, 1], 4, 2, True),
    ("nine taps, ten slabs, several images", (3, 160, 5, 5, 64, 3, 3, 1, 1), [1, 3, 2, 1, 16, 2, 1, 1, 5, 1, 1, 1, 1, 5, 20, 8, 1, 2, 3], 10, 8, True),
    ("nine taps, five slabs of 32 channels", (3, 160, 5, 5, 64, 3, 3, 1, 1), [1, 3, 4, 8, 2, 1, 1, 1, 1, 5, 1, 1, 1, 5, 5, 32, 1, 2, 2], 5, 4, True),
    ("one tap, slabs of 64 channels", (2, 256, 8, 8, 32, 1, 1, 1, 0), [1, 2, 1, 1, 1, 32, 1, 1, 2, 4, 2, 4, 1, 1, 4, 64, 1, 2, 0], 4, 1, False),
    ("two slabs", (1, 32, 8, 8, 32, 1, 1, 1, 0), [1, 1, 1, 1, 4, 8, 1, 1, 4, 2, 1, 4, 1, 2, 16, 2, 1, 2, 3], 2, 1, False),
    ("nine taps, no shared tiles", (3, 160, 5, 5, 64, 3, 3, 1, 1), [1, 3, 1, 1, 8, 8, 1, 5, 1, 1, 1, 5, 1, 1, 5, 32, 1, 2, 0], 5, 1, False),
    ("25 taps", (1, 48, 7, 7, 32, 5, 5, 1, 2), [1, 1, 1, 2, 1, 16, 1, 1, 1, 7, 1, 1, 1, 7, 24, 2, 1, 2, 2], 3, 4, False),
]


@pytest.mark.parametrize("label,dims,cfg,slabs,kw,ahead", CASES, ids=[c[0] for c in CASES])
def test_members(label, dims, cfg, slabs, kw, ahead):
    op = P.opevo_op_create(P.OPEVO_CONV2D, dims, P.OPEVO_F16)
    plan = P.opevo_kernel_plan(op, V, cfg)
    assert plan.status == P.OPEVO_OK and plan.path == 5, plan.reason
    text = P.opevo_kernel_defines(op, V, cfg)
    D = dict(re.findall(r"-D(\w+)=(-?\d+)(?=\s|$)", text))
    assert text.startswith("conv_patch:") and (int(D["KSTEPS"]), int(D["KW"]), D.get("SLABS_AHEAD") == "2") == (slabs, kw, ahead)


@pytest.mark.parametrize("slabs", range(1, 12))
def test_every_pass_multiplies_its_slab(slabs):
    """The order of loads, stores and passes: two register sets and two stages; no slab past the last one is loaded."""
    regs, stage = [0, min(1, slabs - 1)], [0, None]
    done = []
    for s in range(slabs):
        load = s + 2 if s + 2 < slabs else slabs - 1
        assert 0 <= load < slabs
        regs[s & 1] = load
        done.append(stage[s & 1])
        stage[(s + 1) & 1] = regs[(s + 1) & 1]
    assert done == list(range(slabs))


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("label,dims,cfg,slabs,kw,ahead", CASES, ids=[c[0] for c in CASES])
def test_results_match_the_oracle(label, dims, cfg, slabs, kw, ahead, dtype):
    """Products of 16-bit values are exact in fp32; sums of at most 1440 of them, in any order: 1e-5 is 80 roundings."""
    import torch
    from oracle import tensor as T
    img, ker = synth.conv_inputs(*dims[:7], dtype, 7)
    want = T.conv2d(img, ker, dims[7], dims[8]).ravel()
    op = P.opevo_op_create(P.OPEVO_CONV2D, dims, synth.DTYPE_CODE[dtype])
    dk, di = synth.to_device(ker, dtype), synth.to_device(img, dtype)
    dc = torch.full((want.size,), float("nan"), device="cuda:0")
    kernel, _ = P.opevo_kernel_build(op, V, cfg)
    for _ in range(2):                                     # the second launch overwrites what the first one left
        P.opevo_kernel_launch(kernel, dk.data_ptr(), di.data_ptr(), dc.data_ptr(), torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    P.opevo_kernel_destroy(kernel)
    got = dc.cpu().numpy().astype(np.float64)
    assert np.all(np.isfinite(got)) and np.linalg.norm(got - want) <= 1e-5 * np.linalg.norm(want), label
