"""CPU re-computation of the few-channels convolution template (image rows in LDS, taps of a kernel row as the reduction's
groups of 8): every global load lies inside its tensor, every LDS store and fragment read inside the patch and aligned for its
width, boxes are covered once, taps past the kernel are cleared whatever the patch holds there, and the sums the
fragments form are the convolution (direct convolution of integer data, exact) -- for every workgroup, wave, lane, column and step."""
import ctypes
import re

import numpy as np
import pytest

import paper_2006_05664_amd as P
from host_code import compile_common

V4, V4C, V4L, V4P, V4X = P.OPEVO_TILE4, P.OPEVO_TILE4C, P.OPEVO_TILE4L, P.OPEVO_TILE4P, P.OPEVO_TILE4X
CASES = [   # label, dims (B Cin H W Cout Hk Wk stride pad), space, configuration
    ("11x11 stride 4, rows of 7 pixels of 2 images", (2, 3, 35, 35, 32, 11, 11, 4, 0), V4C, [1, 2, 1, 1, 1, 32, 7, 1, 1, 1, 1, 1, 1, 7, 1, 33, 11, 0, 0]),
    ("3x3 padded, stride 1: two copies, 32-row atoms", (1, 3, 9, 12, 32, 3, 3, 1, 1), V4, [1, 1, 1, 1, 1, 32, 3, 1, 1, 3, 2, 1, 1, 6, 3, 9, 1]),
    ("16-row atoms, 5x5, odd width", (1, 1, 11, 13, 16, 5, 5, 1, 2), V4, [1, 1, 1, 1, 1, 16, 11, 1, 1, 1, 1, 1, 1, 13, 1, 25, 0]),
    ("7x7 stride 2, padding 3", (1, 3, 16, 20, 16, 7, 7, 2, 3), V4L, [1, 1, 1, 1, 1, 16, 4, 1, 1, 2, 2, 1, 1, 5, 1, 3, 0, 2, 0]),
    ("image 8 wide, padding wider than a piece is long", (1, 2, 8, 8, 16, 3, 9, 1, 4), V4, [1, 1, 1, 1, 1, 16, 7, 1, 1, 2, 2, 1, 1, 4, 2, 27, 0]),
    ("separately split reduction, stride 3", (1, 2, 14, 17, 32, 3, 2, 3, 0), V4P, [1, 1, 1, 1, 1, 32, 2, 1, 1, 2, 1, 1, 1, 6, 2, 1, 3, 1, 1, 2, 1, 0]),
    ("launch order, two row blocks", (1, 1, 10, 10, 64, 3, 3, 1, 1), V4X, [1, 1, 2, 1, 1, 32, 5, 1, 1, 2, 2, 1, 1, 5, 1, 9, 1, 1, 0, 1]),
]


def _defs(op, variant, cfg):
    text = P.opevo_kernel_defines(op, variant, cfg)
    tmpl, rest = text.split(":", 1)
    return tmpl.strip(), {m.group(1): int(m.group(2)) for m in re.finditer(r"-D(\w+)=(-?\d+)(?=\s|$)", rest)}


def _shift(v, sh):
    out = np.zeros(8)
    n = len(v)
    for i in range(8):
        if 0 <= i + sh < n:
            out[i] = v[i + sh]
    return out


def _direct(img, ker, stride, pad):
    B, C, H, W = img.shape
    M, _, hk, wk = ker.shape
    big = np.zeros((B, C, H + 2 * pad, W + 2 * pad))
    big[:, :, pad:pad + H, pad:pad + W] = img
    ho, wo = (H + 2 * pad - hk) // stride + 1, (W + 2 * pad - wk) // stride + 1
    out = np.zeros((B, M, ho, wo))
    for y in range(ho):
        for x in range(wo):
            out[:, :, y, x] = np.einsum("bcrs,mcrs->bm", big[:, :, y * stride:y * stride + hk, x * stride:x * stride + wk], ker)
    return out


@pytest.mark.parametrize("label,dims,variant,cfg", CASES, ids=[c[0] for c in CASES])
def test_every_address_and_the_sums(label, dims, variant, cfg):
    op = P.opevo_op_create(P.OPEVO_CONV2D, dims, P.OPEVO_BF16)
    plan = P.opevo_kernel_plan(op, variant, cfg)
    tmpl, D = _defs(op, variant, cfg)
    assert plan.status == P.OPEVO_OK and plan.path == 7 and tmpl == "conv_rows" and D["PERSIST"] == 0, (plan.path, plan.reason)
    B, CIN, HIN, WIN, M, HK, WK, S, PAD = dims
    atom, wm_n, wn_n, MI, NI, WKP = D["ATOM"], D["WM"], D["WN"], D["MI"], D["NI"], D["WKP"]
    BM, BN, NB2, BH, BW, H1, W1, HOUT, WOUT, K = (D[k] for k in ("BM", "BN", "NB2", "BH", "BW", "H1", "W1", "HOUT", "WOUT", "K"))
    G, Q = (2 if atom == 32 else 4), WKP // 8
    RPS = G // Q
    SPC = -(-HK // RPS)
    STEPS, PH, PW = CIN * SPC, (BH - 1) * S + HK, (BW - 1) * S + WK
    CPR = -(-PW // 8)
    PITCH, ROWS, ncopy = CPR * 8, NB2 * CIN * PH, 2 if S % 2 else 1
    copy_min = ROWS * PITCH + (SPC * RPS - HK) * PITCH + WKP
    COPY = -(-copy_min // 128) * 128 + 64 if ncopy == 2 else -(-copy_min // 8) * 8
    beside = (BM * K + 128) * 2 if D["STAGE_A"] == 2 else 0           # the kernel tensor's rows
    assert plan.lds_bytes == ncopy * COPY * 2 + beside <= 160 * 1024 and plan.block == 64 * wm_n * wn_n and BM == wm_n * MI * atom and wn_n * NI * atom >= BN
    rng = np.random.default_rng(2)
    img = rng.integers(-4, 5, (B, CIN, HIN, WIN)).astype(float)
    ker = rng.integers(-4, 5, (M, CIN, HK, WK)).astype(float)
    fi, fk = img.ravel(), ker.ravel()
    out = np.full((B, M, HOUT, WOUT), np.nan)
    lanes = np.arange(64)
    for mb in range(M // BM):
        # the kernel tensor's fragments, af[row][step][group] of the rows of this block
        af = np.zeros((BM, STEPS, G, 8))
        for row in range(BM):
            for t in range(STEPS):
                ci, tr = t // SPC, t % SPC * RPS
                for kg in range(G):
                    at = (mb * BM + row) * K + (kg // Q) * WK + kg % Q * 8 + (ci * HK + tr) * WK
                    risky = (ci * HK + tr + RPS - 1) * WK + (Q - 1) * 8 + 8 > K
                    frm = min(at, M * K - 8) if risky else at
                    assert 0 <= frm and frm + 8 <= M * K
                    v = _shift(fk[frm:frm + 8], at - frm) if risky else fk[frm:frm + 8].copy()
                    for i in range(8):
                        if kg % Q * 8 + i >= WK or (t % SPC == SPC - 1 and tr + kg // Q >= HK):
                            v[i] = 0
                    af[row, t, kg] = v
        for box in range(plan.grid[0] * (plan.grid[1] if variant == V4X else 1) // (M // BM if variant == V4X else 1)):
            nb0, y0, x0 = box // (W1 * H1) * NB2, box // W1 % H1 * BH, box % W1 * BW
            patch = np.full(ncopy * COPY, np.nan)
            # the fill's split: threads along a row, several rows at a time -- every piece once, row / PH by a 24-bit multiplication
            NT = plan.block
            TPR, XP = min(CPR, NT), -(-CPR // NT)
            RPP = NT // TPR
            RP = -(-ROWS // RPP)
            seen = np.zeros((ncopy, ROWS, CPR), int)
            for p in range(ncopy * XP * RP):
                for tid in range(TPR * RPP):
                    row, c = tid // TPR + p // XP % RP * RPP, tid % TPR + p % XP * NT
                    assert row * (2 ** 20 // PH + 1) < 2 ** 32 and (PH == 1 or (ROWS + RPP) * PH >= 2 ** 20 or row * (2 ** 20 // PH + 1) >> 20 == row // PH)
                    if row < ROWS and c < CPR:
                        seen[p // (RP * XP), row, c] += 1
            assert (seen == 1).all()
            for q in range(ncopy * ROWS * CPR):
                row, copy, c = q // CPR % ROWS, q // (CPR * ROWS), q % CPR
                x, y = x0 * S - PAD + c * 8 + copy, y0 * S - PAD + row % PH
                xs = min(max(x, 0), WIN - 8)
                v = np.zeros(8)
                if 0 <= y < HIN:
                    at = nb0 * CIN * HIN * WIN + (row // PH * HIN + y) * WIN + xs
                    if PAD == 0:            # what follows the row in memory may stand past its end; the tensor's end is kept
                        at, xs = min(at - xs + x, fi.size - 8), x + min(fi.size - 8 - (at - xs + x), 0)
                    assert 0 <= at and at + 8 <= fi.size
                    v = _shift(fi[at:at + 8], x - xs)
                dst = copy * COPY + row * PITCH + c * 8
                assert dst % 8 == 0 and dst + 8 <= copy * COPY + COPY
                patch[dst:dst + 8] = v
            for col in range(wn_n * NI * atom):
                cn = min(col, BN - 1)
                b, y, xs = cn // (BH * BW), cn // BW % BH, cn % BW * S
                odd = xs & 1 if ncopy == 2 else 0
                acc = np.zeros(BM)
                for t in range(STEPS):
                    off = (t // SPC * PH + t % SPC * RPS) * PITCH
                    for kg in range(G):
                        at = odd * COPY + (b * CIN * PH + y * S + kg // Q) * PITCH + xs - odd + kg % Q * 8 + off
                        assert at % (4 if S % 4 == 0 else 2) == 0 and 0 <= at and at + 8 <= patch.size
                        v = patch[at:at + 8].copy()
                        for i in range(8):
                            if kg % Q * 8 + i >= WK or (t % SPC == SPC - 1 and t % SPC * RPS + kg // Q >= HK):
                                v[i] = 0          # a bitwise and: also for NaN
                        acc += af[:, t, kg] @ v
                if col < BN:
                    bb, yy, xx = nb0 + b, y0 + y, x0 + cn % BW
                    assert np.all(np.isnan(out[bb, mb * BM:(mb + 1) * BM, yy, xx]))
                    out[bb, mb * BM:(mb + 1) * BM, yy, xx] = acc
    assert np.array_equal(out, _direct(img, ker, S, PAD))
    kernel, _ = P.opevo_kernel_build(op, variant, cfg)
    assert 1000 < P.opevo_kernel_code_size(kernel) < (128 << 10)
    P.opevo_kernel_destroy(kernel)


def test_boxes_dealt_to_persistent_workgroups_are_covered_once():
    op = P.opevo_op_create(P.OPEVO_CONV2D, (512, 3, 227, 227, 64, 11, 11, 4, 0), P.OPEVO_BF16)
    cfg = [128, 4, 1, 4, 8, 2, 55, 1, 1, 1, 1, 1, 5, 11, 1, 33, 11, 0, 0]
    plan = P.opevo_kernel_plan(op, V4C, cfg)
    _, D = _defs(op, V4C, cfg)
    assert plan.path == 7 and D["PERSIST"] == plan.grid[0] == 512 and D["NBOX"] == 7040 and plan.grid[1] == plan.grid[2] == 1
    for nbox, persist in ((7040, 512), (2053, 512), (8, 8), (1001, 168), (513, 256)):
        seen = np.zeros(nbox, int)
        per = (nbox + 7) // 8
        for w in range(persist):
            last = min(nbox, (w % 8 + 1) * per)
            for box in range(w % 8 * per + w // 8, last, persist // 8):
                seen[box] += 1
        assert np.all(seen == 1), (nbox, persist)


PLACES = [CASES[0], CASES[1],
          ("eight images of 17 GB of output in a box", (8, 1, 32772, 8, 32768, 5, 5, 1, 0), V4C,
           [1, 8, 512, 2, 1, 32, 32768, 1, 1, 1, 1, 1, 4, 1, 1, 1, 25, 0, 0]),
          ("just below 4 GiB of outputs a box", (7, 1, 3102, 16, 4096, 3, 3, 1, 0), V4, [1, 7, 64, 2, 1, 32, 775, 1, 4, 1, 1, 1, 14, 1, 1, 9, 0])]


@pytest.mark.parametrize("label,dims,variant,cfg", PLACES, ids=[c[0] for c in PLACES])
def test_a_column_s_place_in_the_output(label, dims, variant, cfg):
    """The offset the template stores at, as it is compiled, against the 64-bit index of every (row, column) of a box that begins or ends a range."""
    op = P.opevo_op_create(P.OPEVO_CONV2D, dims, P.OPEVO_BF16)
    plan = P.opevo_kernel_plan(op, variant, cfg)
    assert plan.status == P.OPEVO_OK and plan.path == 7, (plan.path, plan.reason)
    _, D = _defs(op, variant, cfg)
    lib = compile_common(P.opevo_kernel_defines(op, variant, cfg), """
extern "C" unsigned long offset(int m, int c) { return conv_c_offset(m, c); }
extern "C" long wanted(int m, int c) { const ColBlock cb = {0, 0, 0}; return 4 * (conv_c_index(cb, m, c) - conv_c_index(cb, 0, 0)); }
""")
    lib.offset.restype, lib.wanted.restype = ctypes.c_ulong, ctypes.c_long
    box = D["BH"] * D["BW"]
    columns = {b * box + y * D["BW"] + x for b in range(D["NB2"]) for y in {0, D["BH"] - 1} for x in {0, D["BW"] - 1}}
    for c in columns:
        for m in (0, 1, 4, 28):
            assert lib.offset(m, c) == lib.wanted(m, c), (m, c)


def test_which_members_take_the_few_channels_template():
    def path(dims, variant, cfg, dtype=P.OPEVO_BF16):
        plan = P.opevo_kernel_plan(P.opevo_op_create(P.OPEVO_CONV2D, dims, dtype), variant, cfg)
        assert plan.status == P.OPEVO_OK, plan.reason
        return plan.path
    dims, cfg = (1, 3, 9, 12, 32, 3, 3, 1, 1), [1, 1, 1, 1, 1, 32, 3, 1, 1, 3, 2, 1, 1, 6, 3, 9, 1]
    assert path(dims, V4, cfg) == 7 and path(dims, V4, cfg, P.OPEVO_F16) == 7 and path(dims, V4, cfg, P.OPEVO_F32) != 7
    assert path((1, 3, 9, 7, 32, 3, 3, 1, 1), V4, [1, 1, 1, 1, 1, 32, 3, 1, 1, 3, 1, 1, 1, 7, 3, 9, 1]) != 7     # rows shorter than a piece
    assert path(dims, V4, [1, 1, 1, 1, 1, 32, 3, 1, 1, 3, 4, 1, 1, 3, 3, 9, 1]) != 7                              # boxes 3 pixels wide
    assert path(dims, V4C, cfg[:14] + [3, 1, 9, 1, 0]) != 7                                                       # reduction split over workgroups
    assert path((1, 16, 9, 12, 32, 3, 3, 1, 1), V4, [1, 1, 1, 1, 1, 32, 3, 1, 1, 3, 2, 1, 1, 6, 9, 16, 1]) != 7   # 16 channels
    assert path((1, 8, 9, 12, 32, 3, 3, 1, 1), V4C, cfg[:14] + [1, 9, 8, 1, 1]) != 7                              # channels-last copies asked for


GPU_CASES = CASES + [
    ("workgroups that take several boxes, boxes no multiple of eight", (4101, 1, 10, 8, 32, 3, 3, 1, 1), V4, [4101, 1, 1, 1, 1, 32, 1, 1, 10, 1, 1, 1, 8, 1, 1, 9, 0]),
    ("workgroups that take several boxes, two row blocks", (1101, 3, 23, 23, 64, 11, 11, 4, 0), V4, [1101, 1, 2, 1, 1, 32, 4, 1, 1, 1, 1, 1, 4, 1, 3, 121, 0]),
]


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("label,dims,variant,cfg", GPU_CASES, ids=[c[0] for c in GPU_CASES])
def test_results_match_the_oracle(label, dims, variant, cfg, dtype):
    """fp32 sums of at most 363 products of exact inputs: 1e-5 is 80 roundings.  An infinite pixel reaches the outputs whose
    taps touch it and no others, although the patch holds it next to their taps."""
    import torch
    from oracle import tensor as T
    from paper_2006_05664_amd import synth
    img, ker = synth.conv_inputs(*dims[:7], dtype, 5)
    want = T.conv2d(img, ker, dims[7], dims[8])
    op = P.opevo_op_create(P.OPEVO_CONV2D, dims, synth.DTYPE_CODE[dtype])
    assert P.opevo_kernel_plan(op, variant, cfg).path == 7
    assert ("-DPERSIST=0 " in P.opevo_kernel_defines(op, variant, cfg)) == ("several boxes" not in label)
    da, db = synth.to_device(ker, dtype), synth.to_device(img, dtype)
    dc = torch.full((want.size,), float("nan"), device="cuda:0")
    kernel, _ = P.opevo_kernel_build(op, variant, cfg)
    stream = torch.cuda.current_stream().cuda_stream
    P.opevo_kernel_launch(kernel, da.data_ptr(), db.data_ptr(), dc.data_ptr(), stream)
    torch.cuda.synchronize()
    got = dc.cpu().numpy().astype(np.float64)
    assert np.all(np.isfinite(got))
    assert np.linalg.norm(got - want.ravel()) <= 1e-5 * np.linalg.norm(want), label
    place = (dims[0] - 1, 0, dims[2] // 2, dims[3] // 2)
    db[place] = float("inf")
    P.opevo_kernel_launch(kernel, da.data_ptr(), db.data_ptr(), dc.data_ptr(), stream)
    torch.cuda.synchronize()
    P.opevo_kernel_destroy(kernel)
    touched = np.zeros(img.shape)
    touched[place] = 1
    touched = T.conv2d(touched, np.ones_like(ker), dims[7], dims[8]) > 0
    got = dc.cpu().numpy().reshape(want.shape)
    assert np.array_equal(~np.isfinite(got), touched)
