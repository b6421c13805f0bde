"""The ways a ragged MFMA member is built: places of pieces kept where the registers are said to hold them or may hold them, else worked out where they are
needed; what a way without kept places asks the compiler for; results of members on either side of the lines."""
import os
import re
import subprocess

import numpy as np
import pytest

import paper_2006_05664_amd as P
from host_code import CLANG, ROOT
from paper_2006_05664_amd import synth

V = P.OPEVO_TILE4
CASES = [   # label, kind, dims, configuration, waves' atoms, kept places
    ("up to 15 % over, eight waves of 11 x 2 atoms", P.OPEVO_MATMUL, (165, 756, 360), [1, 11, 3, 5, 3, 28, 3, 3, 45, 8, 1], (11, 2), 1),
    ("up to 15 % over, nine waves of 5 x 3", P.OPEVO_MATMUL, (468, 135, 350), [2, 9, 2, 13, 1, 1, 3, 45, 25, 14, 1], (5, 3), 1),
    ("placed piece by piece, eight waves of 1 x 15", P.OPEVO_MATMUL, (126, 950, 420), [6, 1, 3, 7, 1, 38, 5, 5, 28, 15, 1], (1, 15), 0),
    ("placed piece by piece, nine waves of 1 x 11, batches", P.OPEVO_BMM, (12, 144, 165, 180), [6, 2, 1, 72, 1, 2, 1, 5, 11, 3, 5, 36, 0], (1, 11), 0),
    ("worked out for every slab, more rows than columns", P.OPEVO_MATMUL, (400, 2255, 350), [2, 40, 1, 5, 11, 1, 1, 205, 175, 2, 1], (13, 2), 0),
]


def _defs(op, cfg):
    text = P.opevo_kernel_defines(op, V, cfg)
    return text, {m.group(1): int(m.group(2)) for m in re.finditer(r"-D(\w+)=(-?\d+)(?=\s|$)", text)}


@pytest.mark.parametrize("label,kind,dims,cfg,atoms,keep", CASES, ids=[c[0] for c in CASES])
def test_which_way_comes_first_and_that_it_fits(label, kind, dims, cfg, atoms, keep):
    op = P.opevo_op_create(kind, dims, P.OPEVO_BF16)
    plan = P.opevo_kernel_plan(op, V, cfg)
    _, D = _defs(op, cfg)
    assert plan.status == P.OPEVO_OK and plan.path == 6
    assert (D["MI"], D["NI"]) == atoms and D["KEEP"] == keep
    before = P.opevo_code_cache_stats()["misses"]
    kernel, _ = P.opevo_kernel_build(op, V, cfg)
    P.opevo_kernel_destroy(kernel)
    assert P.opevo_code_cache_stats()["misses"] - before == 1, "the first way spills"


@pytest.mark.parametrize("keep", [0, 1])
def test_without_kept_places_nothing_is_asked_for_a_second_workgroup(keep):
    """4 waves that are to share a compute unit's registers with another workgroup when places are kept (two waves a SIMD): not when they are not."""
    op = P.opevo_op_create(P.OPEVO_MATMUL, (1250, 2440, 783), P.OPEVO_F16)
    text, D = _defs(op, [50, 5, 5, 1, 40, 1, 61, 1, 29, 27, 1])
    assert D["NT"] == 256 and D["KEEP"] == 1 and D["MINW"] == 2 and D["DEPTH"] == 1
    macros = [o for o in text.split(":", 1)[1].split() if not o.startswith("-DKEEP")] + ["-DKEEP=%d" % keep] + ([] if keep else ["-DFRESH=1"])
    src = os.path.join(ROOT, "paper_2006_05664_amd", "csrc", "templates", "gemm_ragged.hip")
    out = subprocess.run([CLANG, "-E", "-P", "-x", "c++", src] + macros, capture_output=True, text=True, check=True).stdout
    threads, waves = re.search(r"__launch_bounds__\(([^,]+),\s*(.+)\)\s*void", out).groups()
    assert eval(threads) == 256 and eval(waves.replace("/", "//")) == (2 if keep else 1)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("label,kind,dims,cfg,atoms,keep", CASES, ids=[c[0] for c in CASES])
def test_results_match_the_oracle(label, kind, dims, cfg, atoms, keep, dtype):
    """Products of 16-bit values are exact in fp32; sums of at most 420 of them: 1e-5 is 80 roundings."""
    import torch
    from oracle import tensor as T
    a, b = (synth.matmul_inputs if kind == P.OPEVO_MATMUL else synth.bmm_inputs)(*dims, dtype, 5)
    want = (T.matmul(a, b) if kind == P.OPEVO_MATMUL else T.bmm(a, b)).ravel()
    op = P.opevo_op_create(kind, dims, synth.DTYPE_CODE[dtype])
    dc = torch.full((want.size,), float("nan"), device="cuda:0")
    da, db = synth.to_device(a, dtype), synth.to_device(b, dtype)
    kernel, _ = P.opevo_kernel_build(op, V, cfg)
    for _ in range(2):
        P.opevo_kernel_launch(kernel, da.data_ptr(), db.data_ptr(), dc.data_ptr(), torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    P.opevo_kernel_destroy(kernel)
    got = dc.cpu().numpy().astype(np.float64)
    assert np.all(np.isfinite(got)) and np.linalg.norm(got - want) <= 1e-5 * np.linalg.norm(want), label
