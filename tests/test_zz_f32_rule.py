"""Which fp32 members have the pipelined slab loop: two-stage ones, but not short reductions on a full chip and not
convolutions on slabs of one group of 8."""
import pytest

import paper_2006_05664_amd as P

MM, BMM, TA, CONV = P.OPEVO_MATMUL, P.OPEVO_BMM, P.OPEVO_BMM_TA, P.OPEVO_CONV2D


def _pipelined(kind, dims, cfg):
    op = P.opevo_op_create(kind, dims, P.OPEVO_F32)
    plan = P.opevo_kernel_plan(op, P.OPEVO_TILE4, cfg)
    assert plan.status == P.OPEVO_OK and plan.path == 4, (plan.path, plan.reason)
    return "-DPIPELINED=1" in P.opevo_kernel_defines(op, P.OPEVO_TILE4, cfg).split()


def test_the_options_say_which_loop_a_member_has():
    assert _pipelined(MM, (512, 4096, 1024), [8, 2, 16, 2, 64, 2, 32, 1, 16, 64, 1])
    assert not _pipelined(MM, (512, 4096, 1024), [8, 2, 16, 2, 64, 2, 32, 1, 16, 64, 0])       # one stage
    assert not _pipelined(TA, (960, 128, 64, 128), [960, 1, 1, 2, 2, 32, 1, 2, 1, 32, 4, 32, 1])   # 960 x 4 waves, 4 slabs


@pytest.mark.parametrize("kind,dims,cfg,want", [
    (MM, (2048, 2048, 128), [32, 1, 1, 64, 32, 2, 1, 32, 16, 8, 1], False),      # 1024 x 2 waves, 16 slabs of 8: 15.7 against 17.5 us
    (MM, (2048, 2048, 256), [32, 1, 1, 64, 32, 2, 1, 32, 32, 8, 1], True),       # a longer reduction
    (MM, (1024, 1024, 128), [16, 1, 1, 64, 16, 2, 1, 32, 16, 8, 1], True),       # the chip not full
    (CONV, (8, 64, 28, 28, 64, 3, 3, 1, 1), [8, 1, 1, 1, 1, 64, 14, 1, 1, 2, 1, 1, 1, 28, 72, 8, 1], False),   # slabs of one group, gathered
    (CONV, (8, 64, 28, 28, 64, 3, 3, 1, 1), [8, 1, 1, 1, 1, 64, 14, 1, 1, 2, 1, 1, 1, 28, 36, 16, 1], True),
    (CONV, (8, 64, 28, 28, 64, 3, 3, 1, 1), [8, 1, 1, 1, 1, 64, 14, 1, 1, 2, 1, 1, 1, 28, 64, 9, 1], True),    # padded to 16
])
def test_members_that_the_pipelined_loop_slows_down_keep_the_plain_one(kind, dims, cfg, want):
    assert _pipelined(kind, dims, cfg) == want
