"""Conv2d members on the row-strip template (csrc/templates/conv_strip.hip): which members run there, and the kernel computed again on the
CPU from the constants the decoder hands it, thread by thread -- every global access inside its tensor, every LDS access inside its part, every value
in its place, and the sum the fragments form compared with a direct convolution (integer data: exact).  The GPU tests compare the results with the
oracle."""
import re

import numpy as np
import pytest

import paper_2006_05664_amd as P
from paper_2006_05664_amd import synth

V = P.OPEVO_TILE4L

CASES = [   # label, dims (B, Cin, H, W, Cout, Hk, Wk, stride, pad), dtype, configuration, what the decoder must choose
    ("3x3, one strip, 7 rows a wave", (2, 64, 14, 14, 64, 3, 3, 1, 1), "bf16", [2, 1, 1, 2, 1, 32, 1, 7, 2, 1, 1, 1, 14, 1, 4, 16, 0, 2, 0], dict(ATOM=16)),
    ("3x3, two strips of a 28-wide row, slabs of one tap group", (2, 32, 28, 28, 64, 3, 3, 1, 1), "f16", [2, 1, 1, 2, 1, 32, 4, 7, 1, 1, 1, 1, 28, 1, 2, 16, 0, 2, 0], dict(ATOM=16)),
    ("3x3, odd width, 27 of 32 lanes", (3, 32, 27, 27, 64, 3, 3, 1, 1), "bf16", [3, 1, 1, 2, 1, 32, 9, 3, 1, 1, 1, 1, 27, 1, 2, 16, 0, 2, 0], dict(ATOM=16, R=3)),
    ("5x5, boxes of half a row, 16 channels", (1, 16, 56, 56, 64, 5, 5, 1, 2), "bf16", [1, 1, 1, 2, 1, 32, 7, 4, 2, 1, 2, 1, 28, 1, 1, 16, 0, 2, 0], dict(ATOM=32, CS=16)),
    ("5x5, odd width, two images a box (folded)", (4, 64, 27, 27, 64, 5, 5, 1, 2), "bf16", [2, 2, 1, 1, 32, 2, 3, 3, 1, 3, 1, 9, 1, 3, 16, 4, 0, 2, 1], dict(NB2=2)),
    ("3x3, a whole image a box (folded)", (2, 256, 14, 14, 64, 3, 3, 1, 1), "bf16", [2, 1, 2, 1, 8, 4, 1, 7, 2, 1, 1, 14, 1, 1, 8, 32, 0, 2, 1], dict(ATOM=16)),
    ("3x3, odd width, three waves share a wave tile", (1, 128, 27, 27, 32, 3, 3, 1, 1), "f16", [1, 1, 1, 1, 1, 32, 9, 3, 1, 1, 1, 1, 27, 1, 8, 16, 0, 2, 0], dict(KW=3)),
    ("1x1, two rows a wave", (4, 64, 14, 14, 64, 1, 1, 1, 0), "bf16", [4, 1, 1, 2, 1, 32, 1, 7, 2, 1, 1, 1, 14, 1, 4, 16, 0, 2, 0], dict(CS=64)),
    ("3x3 without padding, wider image than output", (2, 32, 16, 16, 64, 3, 3, 1, 0), "bf16", [2, 1, 1, 2, 1, 32, 1, 7, 2, 1, 1, 1, 14, 1, 2, 16, 0, 2, 0], dict(ATOM=16)),
    ("1x9, 48 output channels", (2, 32, 8, 36, 48, 1, 9, 1, 0), "bf16", [2, 1, 1, 3, 1, 16, 1, 8, 1, 1, 1, 1, 28, 1, 1, 32, 0, 2, 0], dict(WM=3)),
    ("3x3, two waves share a tile of seven atoms: the final sum in passes of six and one", (2, 256, 14, 14, 64, 3, 3, 1, 1), "bf16",
     [1, 2, 2, 2, 1, 16, 1, 7, 2, 1, 1, 1, 1, 14, 8, 32, 1, 2, 1], dict(KW=2, MI=1, R=7, LDS_BYTES=103424)),
    ("3x3, odd width, three waves, nine atoms in three passes of three", (2, 64, 27, 27, 32, 3, 3, 1, 1), "f16",
     [2, 1, 1, 4, 1, 8, 3, 1, 3, 3, 1, 9, 1, 3, 32, 2, 0, 2, 1], dict(KW=3, R=9, LDS_BYTES=41984)),
    ("3x3, six waves, fourteen atoms in passes of five", (2, 128, 14, 14, 32, 3, 3, 1, 1), "bf16",
     [2, 1, 1, 1, 32, 1, 1, 7, 1, 2, 1, 14, 1, 1, 32, 4, 1, 2, 3], dict(KW=6, LDS_BYTES=70656)),
    ("5x3, 12 columns of 14 pixels", (2, 32, 12, 14, 48, 5, 3, 1, 1), "bf16", [2, 1, 1, 3, 1, 16, 1, 2, 5, 1, 1, 1, 14, 1, 1, 32, 0, 2, 0], dict(WM=3, R=2)),
]
# members of the same space that keep the patch template
STAY = [
    ("flag 1 asks for the two-stage loop", (2, 64, 14, 14, 64, 3, 3, 1, 1), [2, 1, 1, 2, 1, 32, 1, 7, 2, 1, 1, 1, 14, 1, 4, 16, 1, 2, 0]),
    ("asks for two waves per tile", (2, 64, 14, 14, 64, 3, 3, 1, 1), [2, 1, 2, 1, 1, 32, 1, 7, 2, 1, 1, 1, 14, 1, 4, 16, 0, 2, 1]),
    ("rows of 11 pixels fill less than four lanes of five", (2, 64, 11, 11, 64, 3, 3, 1, 1), [2, 1, 2, 1, 1, 32, 1, 11, 1, 1, 1, 1, 11, 1, 2, 32, 0, 2, 0]),
    ("stride 2", (2, 64, 28, 28, 64, 3, 3, 2, 1), [2, 1, 1, 2, 1, 32, 1, 7, 2, 1, 1, 1, 14, 1, 4, 16, 0, 2, 0]),
]


def _defs(op, cfg):
    tmpl, rest = P.opevo_kernel_defines(op, V, cfg).split(":", 1)
    return tmpl, {m.group(1): int(m.group(2)) for m in (re.match(r"-D(\w+)=(-?\d+)$", t) for t in rest.split()) if m}


def _final_sum(D):
    """The partial sums of KW waves by way of LDS: every place lies inside it, a pass reads what it wrote, every atom is stored once.  Returns the
    atoms a pass takes and those a wave has."""
    Q, atoms, tiles, KW = (4 if D["ATOM"] == 32 else 1), D["MI"] * D["R"], D["WM"] * D["WN"], D["KW"]
    waves = tiles * KW
    per_pass = min(D["LDS_BYTES"] // (waves * Q * 1024), atoms)
    assert per_pass >= 1
    lane = np.arange(64)
    stored = np.zeros((tiles, atoms), dtype=int)
    for a0 in range(0, atoms, per_pass):
        held = np.full(D["LDS_BYTES"] // 16, -1, dtype=np.int64)        # who wrote a place in this pass: ((wave, atom), quarter, lane)
        name = lambda wave, a, q: ((wave * atoms + a) * Q + q) * 64 + lane
        here = range(a0, min(a0 + per_pass, atoms))
        for wave in range(waves):
            for a in here:
                for q in range(Q):
                    at = (((a - a0) * waves + wave) * Q + q) * 64 + lane
                    assert (at < held.size).all() and (held[at] == -1).all()
                    held[at] = name(wave, a, q)
        for wave in range(waves):
            wk, tile = wave // tiles, wave % tiles
            for a in range(a0 + wk, here.stop, KW):
                stored[tile, a] += 1
                for q in range(Q):
                    for k in range(KW):
                        assert (held[(((a - a0) * waves + k * tiles + tile) * Q + q) * 64 + lane] == name(k * tiles + tile, a, q)).all()
    assert (stored == 1).all()
    return per_pass, atoms


def _emulate(dims, cfg, img=None, ker=None, blocks=None):
    """Plays the kernel of the given workgroups (all by default); with operands, returns the output."""
    nimg, cin, hin, win, cout, hk, wk, _, pad = dims
    op = P.opevo_op_create(P.OPEVO_CONV2D, dims, P.OPEVO_BF16)
    plan = P.opevo_kernel_plan(op, V, cfg)
    tmpl, D = _defs(op, cfg)
    assert plan.status == P.OPEVO_OK and plan.path == 5 and tmpl == "conv_strip", (plan.status, plan.path, tmpl)
    BM, BH, BW, NB2, CS, ATOM, WM, WN, MI, R, KW, PWP, NT, H1, W1 = (D[k] for k in "BM BH BW NB2 CS ATOM WM WN MI R KW PWP NT H1 W1".split())
    T, PH, PW, SPR, RG, NCH = hk * wk, BH + hk - 1, BW + wk - 1, -(-BW // ATOM), BH // R, CS // 8
    wk_n, KA, NACC = wk, *((16, 16) if ATOM == 32 else (32, 4))
    KKS, HOUT, WOUT = CS // KA, D["HOUT"], D["WOUT"]
    P_STAGE, A_STAGE = NB2 * PH * PWP * CS, T * BM * CS
    STAGE, UNITS = P_STAGE + A_STAGE, KKS * wk
    assert NT == plan.block == 64 * WM * WN * KW <= 1024 and WN == NB2 * SPR * RG and BM == WM * MI * ATOM and BH == R * RG and UNITS % KW == 0
    assert PWP >= PW and PWP % 16 == 0 and cin % CS == 0 and D["KSTEPS"] * CS == cin
    assert (STAGE + 512) * 2 <= D["LDS_BYTES"] == plan.lds_bytes <= 160 * 1024 and MI * R * NACC == plan.acc_per_lane <= 256
    assert plan.grid[0] * NB2 * BH * BW == nimg * HOUT * WOUT and plan.grid[1] * BM == cout and plan.grid[2] == 1
    aligned = win % 2 == 0
    if KW > 1:
        _final_sum(D)

    def swz(p):
        if NCH == 16:
            return p & 15 if ATOM == 32 else (p & 7) * 2
        return (p // (16 // NCH)) % NCH if ATOM == 32 else ((p // (16 // NCH)) % (NCH // 2)) * 2

    inx, iny = min(PW - pad, win), min(PH - pad, hin)
    npair = (inx + 1) // 2 if W1 == 1 else PW // 2 + 1
    nrow = iny if H1 == 1 else PH
    pairs = npair * nrow * NB2
    tid = np.arange(NT)
    have = img is not None
    out = np.full((nimg, cout, HOUT, WOUT), np.nan)
    written = np.zeros(out.shape, dtype=np.int64)
    lane = np.arange(64)
    lrow, kc = lane % ATOM, lane // ATOM
    for bx, by in blocks or [(x, y) for x in range(plan.grid[0]) for y in range(plan.grid[1])]:
        x0, y0, nb0, m0 = (bx % W1) * BW, ((bx // W1) % H1) * BH, (bx // (W1 * H1)) * NB2, by * BM
        yin0, xin0 = y0 - pad, x0 - pad
        src = np.full(STAGE + 512, -1, dtype=np.int64)        # which element of the image, then of the kernel tensor, a place holds (slab 0)
        hits = np.zeros(STAGE + 512, dtype=np.int64)
        for i in range(-(-NCH * pairs // NT)):
            q = tid + i * NT
            c, pr = q // pairs, q % pairs
            jp, b = pr % npair, pr // (npair * nrow)
            y = (0 if H1 == 1 else yin0) + (pr // npair) % nrow
            x = (0 if W1 == 1 else xin0 & ~1) + 2 * jp
            py, px = y - yin0, x - xin0
            inside = (q < NCH * pairs) & (y >= 0) & (y < hin) & (x >= 0) & (x < win)
            v0 = inside & (px >= 0) & (px < PW)
            v1 = inside & (px + 1 >= 0) & (px + 1 < PW) & (aligned | (x + 1 < win))
            left = np.where((not aligned) & (x == win - 1), 1, 0)
            at = np.where(v0 | v1, (((nb0 + b) * cin + 8 * c) * hin + y) * win + x - left, 0)
            lf = np.where(v0 | v1, left, 0)
            for s in (0, D["KSTEPS"] - 1):
                for ch in range(8):
                    e = at + (s * CS + ch) * hin * win
                    assert (e >= 0).all() and (e + 2 <= img_elems(dims)).all() and (not aligned or (e % 2 == 0).all()), "image load"
            p = (b * PH + py) * PWP + px
            for v, pp, e in ((v0, p, 0), (v1, p + 1, 1)):
                dst = np.where(v, pp * NCH + (c ^ swz(pp)), STAGE // 8 + (tid & 63))
                assert (dst >= 0).all() and (dst * 8 + 8 <= STAGE + 512).all() and (dst[v] * 8 + 8 <= P_STAGE).all(), "image store"
                for ch in range(8):
                    np.add.at(hits, dst[v] * 8 + ch, 1)
                    assert (e + lf[v] <= 1).all()
                    src[dst[v] * 8 + ch] = at[v] + ch * hin * win + e + lf[v]
        for i in range(-(-BM * CS // 2 // NT)):
            q = tid + i * NT
            on = q < BM * CS // 2
            cp, m = q % (CS // 2), q // (CS // 2)
            at = np.where(on, (m0 + m) * cin * T + 2 * cp * T, 0)
            assert (at % 2 == 0).all() and (at + ((D["KSTEPS"] - 1) * CS + 2) * T <= cout * cin * T).all(), "kernel-tensor load"
            for t in range(T):
                w = P_STAGE // 2 + m * (CS // 2) + (((cp >> 2) ^ swz(m)) << 2) + (cp & 3) + t * (BM * CS // 2)
                assert (2 * w[on] >= P_STAGE).all() and (2 * w[on] + 2 <= STAGE).all(), "kernel-tensor store"
                for ch in range(2):
                    np.add.at(hits, 2 * w[on] + ch, 1)
                    src[2 * w[on] + ch] = at[on] + ch * T + t
        assert hits[:STAGE].max() == 1 and (hits[P_STAGE:STAGE] == 1).all(), "an LDS place is written twice, or a kernel-tensor place not at all"
        for b in range(NB2):
            for py in range(PH):
                for px in range(PWP):
                    y, x, p = yin0 + py, xin0 + px, (b * PH + py) * PWP + px
                    if 0 <= y < hin and 0 <= x < win and px < PW:
                        ch = np.arange(CS)
                        place = p * CS + (((ch >> 3) ^ swz(p)) << 3) + (ch & 7)
                        assert (src[place] == (((nb0 + b) * cin + ch) * hin + y) * win + x).all(), ("patch", b, py, px)
                    else:
                        assert (hits[p * CS:(p + 1) * CS] == 0).all(), "a place outside the image is written"
        for wave in range(WM * WN):
            wm, wn = wave // WN, wave % WN
            im, strip, rg = wn // (SPR * RG), wn // RG % SPR, wn % RG
            xl = strip * ATOM + lrow
            pix = (im * PH + rg * R) * PWP + np.minimum(xl, BW - 1)
            acc = np.zeros((MI, R, ATOM, ATOM))
            done = np.zeros((MI, R, T, KKS), dtype=np.int64)
            for wk in range(KW):
                for u in range(wk, UNITS, KW):
                    kk, s = u // wk_n, u % wk_n
                    c, p = kk * (KA // 8) + kc, pix + s
                    a_at = P_STAGE + (wm * MI * ATOM + lrow) * CS + ((c ^ swz(lrow)) << 3) + s * BM * CS
                    p_at = p * CS + ((c ^ swz(p)) << 3)
                    for y in range(R + hk - 1):
                        bo = p_at + y * PWP * CS
                        assert (bo % 8 == 0).all() and (bo >= 0).all() and (bo + 8 <= P_STAGE).all(), "image fragment"
                        for r in range(hk):
                            if not 0 <= y - r < R:
                                continue
                            for i in range(MI):
                                ao = a_at + (r * wk_n * BM + i * ATOM) * CS
                                assert (ao % 8 == 0).all() and (ao >= P_STAGE).all() and (ao + 8 <= STAGE).all(), "kernel fragment"
                                done[i, y - r, r * wk_n + s, kk] += 1
                                for slab in range(D["KSTEPS"] if have else 0):
                                    e = np.arange(8)
                                    sa, sb = src[ao[:, None] + e], src[bo[:, None] + e]
                                    av = ker.reshape(-1)[sa + slab * CS * T]
                                    bv = np.where(sb >= 0, img.reshape(-1)[np.maximum(sb, 0) + slab * CS * hin * win], 0.0)
                                    for g in range(64 // ATOM):
                                        sel = slice(g * ATOM, (g + 1) * ATOM)
                                        acc[i, y - r] += av[sel] @ bv[sel].T
            assert (done == 1).all(), "an MFMA step is missing or taken twice"
            for i in range(MI):
                for j in range(R):
                    cols = np.arange(ATOM)[strip * ATOM + np.arange(ATOM) < BW]
                    rows = m0 + (wm * MI + i) * ATOM + np.arange(ATOM)
                    yy, xx = y0 + rg * R + j, x0 + strip * ATOM + cols
                    written[nb0 + im, rows[:, None], yy, xx[None, :]] += 1
                    if have:
                        out[nb0 + im, rows[:, None], yy, xx[None, :]] = acc[i, j][:, cols]
    return out, written


def img_elems(dims):
    return dims[0] * dims[1] * dims[2] * dims[3]


def _direct(img, ker, pad):
    n, cin, h, w = img.shape
    cout, _, hk, wk = ker.shape
    padded = np.pad(img, ((0, 0), (0, 0), (pad, pad), (pad, pad)))
    ho, wo = h + 2 * pad - hk + 1, w + 2 * pad - wk + 1
    out = np.zeros((n, cout, ho, wo))
    for r in range(hk):
        for s in range(wk):
            out += np.tensordot(ker[:, :, r, s], padded[:, :, r:r + ho, s:s + wo], axes=(1, 1)).transpose(1, 0, 2, 3)
    return out


@pytest.mark.parametrize("label,dims,dtype,cfg,want", CASES, ids=[c[0] for c in CASES])
def test_the_template_computes_the_convolution(label, dims, dtype, cfg, want):
    _, D = _defs(P.opevo_op_create(P.OPEVO_CONV2D, dims, synth.DTYPE_CODE[dtype]), cfg)
    assert {k: D[k] for k in want} == want, D
    rng = np.random.default_rng(3)
    img = rng.integers(-3, 4, size=dims[:4]).astype(np.float64)
    ker = rng.integers(-3, 4, size=(dims[4], dims[1]) + dims[5:7]).astype(np.float64)
    small = img_elems(dims) * dims[4] * dims[5] * dims[6] <= 3e7
    if small:
        out, written = _emulate(dims, cfg, img, ker)
        assert (written == 1).all() and np.array_equal(out, _direct(img, ker, dims[8]))
    else:
        _, written = _emulate(dims, cfg)
        assert (written == 1).all()


def test_final_sums_of_one_and_of_several_passes():
    passes = set()
    for label, dims, dtype, cfg, _ in CASES:
        _, D = _defs(P.opevo_op_create(P.OPEVO_CONV2D, dims, synth.DTYPE_CODE[dtype]), cfg)
        if D["KW"] > 1:
            per_pass, atoms = _final_sum(D)
            passes.add("one" if per_pass == atoms else "even" if atoms % per_pass == 0 else "uneven")
    assert passes == {"one", "even", "uneven"}


@pytest.mark.parametrize("label,dims,cfg", STAY, ids=[c[0] for c in STAY])
def test_members_that_keep_the_patch_template(label, dims, cfg):
    op = P.opevo_op_create(P.OPEVO_CONV2D, dims, P.OPEVO_BF16)
    assert P.opevo_kernel_plan(op, V, cfg).path == 5 and _defs(op, cfg)[0] == "conv_patch"


def test_random_members_stay_in_bounds_and_cover_their_output_once():
    """Members of five operators as a search draws them (folded ones among them): corner and inner workgroups."""
    rng, seen = np.random.default_rng(5), 0
    for dims in ((32, 256, 14, 14, 256, 3, 3, 1, 1), (64, 64, 28, 28, 128, 3, 3, 1, 1), (6, 64, 27, 27, 96, 5, 5, 1, 2), (100, 128, 14, 14, 64, 1, 1, 1, 0),
                 (4, 32, 13, 13, 64, 3, 3, 1, 1)):
        op = P.opevo_op_create(P.OPEVO_CONV2D, dims, P.OPEVO_BF16)
        sp, g = P.opevo_op_space(op, V), P.opevo_rng_create(int(rng.integers(1 << 30)))
        found = 0
        for _ in range(6000):
            cfg = [int(v) for v in P.opevo_space_random(sp, g)]
            if cfg[17] != 2 or P.opevo_kernel_plan(op, V, cfg).status != P.OPEVO_OK or _defs(op, cfg)[0] != "conv_strip":
                continue
            plan = P.opevo_kernel_plan(op, V, cfg)
            gx, gy = plan.grid[0], plan.grid[1]
            _emulate(dims, cfg, blocks=sorted({(x, y) for x in (0, gx - 1) for y in (0, gy - 1)})[:2])
            found += 1
            if found == 4:
                break
        seen += found
        P.opevo_rng_destroy(g); P.opevo_space_destroy(sp)
    assert seen >= 15


@pytest.mark.gpu
@pytest.mark.parametrize("label,dims,dtype,cfg,want", CASES, ids=[c[0] for c in CASES])
def test_results_match_the_oracle(label, dims, dtype, cfg, want):
    """Products of 16-bit values are exact in fp32; sums of at most 2304 of them in some order: 1e-5 is 80 roundings."""
    import torch
    from oracle import tensor as T
    x, w = synth.conv_inputs(*dims[:7], dtype, 5)
    ref = T.conv2d(x, w, dims[7], dims[8])
    op = P.opevo_op_create(P.OPEVO_CONV2D, dims, synth.DTYPE_CODE[dtype])
    dx, dw = synth.to_device(x, dtype), synth.to_device(w, dtype)
    dy = torch.full((ref.size,), float("nan"), device="cuda:0")
    kernel, _ = P.opevo_kernel_build(op, V, cfg)
    for _ in range(3):
        P.opevo_kernel_launch(kernel, dw.data_ptr(), dx.data_ptr(), dy.data_ptr(), torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    P.opevo_kernel_destroy(kernel)
    got = dy.cpu().numpy().astype(np.float64)
    assert np.all(np.isfinite(got)) and np.linalg.norm(got - ref.ravel()) <= 1e-5 * np.linalg.norm(ref), label
