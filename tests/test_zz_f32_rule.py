"""Which loop the two-stage fp32 members are compiled with: the pipelined one, the plain one for short reductions on a full chip, the
plain one with step-by-step reads for convolutions (and those short reductions) on slabs of one group of 8; and that a member whose
kernel spills registers with its loop has another."""
import re
import subprocess

import pytest

import paper_2006_05664_amd as P

MM, BMM, TA, CONV = P.OPEVO_MATMUL, P.OPEVO_BMM, P.OPEVO_BMM_TA, P.OPEVO_CONV2D


def _loop(kind, dims, cfg):
    op = P.opevo_op_create(kind, dims, P.OPEVO_F32)
    plan = P.opevo_kernel_plan(op, P.OPEVO_TILE4, cfg)
    assert plan.status == P.OPEVO_OK and plan.path == 4, (plan.path, plan.reason)
    words = P.opevo_kernel_defines(op, P.OPEVO_TILE4, cfg).split()
    if words[0] != "gemm_mfma_f32:":
        return words[0]
    return "pipelined" if "-DPIPELINED=1" in words else "step" if "-DSTEP_READS=1" in words else "plain"


@pytest.mark.parametrize("kind,dims,cfg,want", [
    (MM, (512, 4096, 1024), [8, 2, 16, 2, 64, 2, 32, 1, 16, 64, 1], "gemm_f32_split:"),     # another template, with a loop of its own
    (MM, (512, 4032, 1024), [8, 2, 16, 2, 42, 1, 96, 1, 16, 64, 1], "pipelined"),           # 96 columns
    (TA, (4, 64, 128, 448), [2, 2, 1, 2, 1, 32, 2, 2, 1, 32, 14, 32, 1], "pipelined"),
    (MM, (512, 4096, 1024), [8, 2, 16, 2, 64, 2, 32, 1, 16, 64, 0], "plain"),           # one stage
    (TA, (960, 128, 64, 128), [960, 1, 1, 2, 2, 32, 1, 2, 1, 32, 4, 32, 1], "plain"),   # 960 x 4 waves, 4 slabs
    (MM, (2048, 2048, 128), [32, 1, 1, 64, 32, 2, 1, 32, 16, 8, 1], "step"),            # 1024 x 2 waves, 16 slabs of 8: 15.7 us; pipelined 17.5
    (MM, (2048, 2048, 256), [32, 1, 1, 64, 32, 2, 1, 32, 32, 8, 1], "pipelined"),       # a longer reduction
    (MM, (1024, 1024, 128), [16, 1, 1, 64, 16, 2, 1, 32, 16, 8, 1], "pipelined"),       # the chip not full
    (CONV, (8, 64, 28, 28, 64, 3, 3, 1, 1), [8, 1, 1, 1, 1, 64, 14, 1, 1, 2, 1, 1, 1, 28, 72, 8, 1], "step"),
    (CONV, (8, 64, 28, 28, 64, 3, 3, 1, 1), [8, 1, 1, 1, 1, 64, 14, 1, 1, 2, 1, 1, 1, 28, 36, 16, 1], "pipelined"),
    (CONV, (8, 64, 28, 28, 64, 3, 3, 1, 1), [8, 1, 1, 1, 1, 64, 14, 1, 1, 2, 1, 1, 1, 28, 64, 9, 1], "pipelined"),    # padded to 16
])
def test_which_loop_a_member_has(kind, dims, cfg, want):
    assert _loop(kind, dims, cfg) == want


@pytest.mark.parametrize("dims,cfg", [     # 16 and 12 bytes of scratch with step-by-step reads, none with the pipelined loop (hipRTC 7.2; 7.0: 12 with any for the second)
    ((8, 64, 28, 28, 64, 3, 3, 1, 1), [4, 2, 1, 1, 2, 32, 1, 1, 1, 28, 2, 14, 1, 1, 96, 6, 1]),
    ((16, 32, 27, 27, 96, 5, 5, 1, 2), [8, 2, 1, 1, 12, 8, 3, 1, 9, 1, 1, 9, 3, 1, 160, 5, 1]),
])
def test_a_member_whose_loop_spills_has_another(dims, cfg, tmp_path):
    op = P.opevo_op_create(CONV, dims, P.OPEVO_F32)
    assert _loop(CONV, dims, cfg) == "step"
    P.opevo_code_cache_configure(str(tmp_path), 0)          # the cache's directory: where the code objects can be read
    try:
        kernel, _ = P.opevo_kernel_build(op, P.OPEVO_TILE4, cfg)
        P.opevo_kernel_destroy(kernel)
    finally:
        P.opevo_code_cache_configure(None, 256 << 20)
    scratch = []            # in the order of the compilations
    for i, entry in enumerate(sorted(tmp_path.iterdir(), key=lambda f: f.stat().st_mtime_ns)):
        data = entry.read_bytes()
        code = tmp_path.parent / ("kernel%d.co" % i)
        code.write_bytes(data[data.index(b"\x7fELF"):])
        notes = subprocess.run(["/opt/rocm/llvm/bin/llvm-readelf", "--notes", str(code)], capture_output=True, text=True, check=True).stdout
        scratch.append(int(re.search(r"private_segment_fixed_size:\s+(\d+)", notes)[1]))
    assert all(scratch[:-1]) and (scratch[-1] == 0 or len(scratch) == 3), scratch
