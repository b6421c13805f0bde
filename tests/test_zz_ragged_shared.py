"""Ragged MFMA members whose waves share the reduction: which they are; every global load inside its operand, every LDS access inside the wave's part, and
fragments that hold the operands' values, each reduction position once (re-computed on the CPU); results where tiles, tails and row ends meet."""
import re

import numpy as np
import pytest

import paper_2006_05664_amd as P
from paper_2006_05664_amd import synth

MM, BMM, TA = P.OPEVO_MATMUL, P.OPEVO_BMM, P.OPEVO_BMM_TA
V, X, K3 = P.OPEVO_TILE4, P.OPEVO_TILE4X, P.OPEVO_TILE4K
CASES = [   # label, kind, dims, variant, configuration, waves that share the reduction (0: the slab walk)
    ("every extent odd, a tail of 9", MM, (63, 105, 457), V, [3, 1, 1, 21, 3, 1, 1, 35, 457, 1, 1], 8),
    ("no tail, 15 columns", MM, (60, 45, 480), V, [2, 1, 1, 30, 3, 1, 1, 15, 15, 32, 1], 8),
    ("the shortest reduction, 3 columns: several tiles begin further left", MM, (32, 33, 448), V, [2, 1, 1, 16, 11, 1, 1, 3, 14, 32, 1], 8),
    ("a shorter one", MM, (32, 33, 447), V, [2, 1, 1, 16, 11, 1, 1, 3, 149, 3, 1], 0),
    ("one tile along a row of 27", MM, (40, 27, 450), V, [2, 1, 1, 20, 1, 1, 1, 27, 15, 30, 1], 8),
    ("first operand transposed, both begin further left", TA, (3, 54, 70, 495), V, [3, 1, 2, 1, 1, 27, 2, 1, 1, 35, 9, 55, 1], 8),
    ("first operand transposed, one tile either way", TA, (2, 27, 35, 450), V, [2, 1, 1, 1, 1, 27, 1, 1, 1, 35, 10, 45, 1], 8),
    ("several batches a workgroup", BMM, (6, 25, 40, 550), V, [2, 3, 1, 1, 1, 25, 1, 1, 1, 40, 11, 50, 1], 8),
    ("launch order", MM, (72, 55, 640), X, [4, 1, 1, 18, 5, 1, 1, 11, 20, 32, 1, 1, 0, 2], 8),
    ("a long reduction", MM, (54, 60, 1310), V, [2, 1, 1, 27, 2, 1, 1, 30, 131, 10, 1], 8),
    ("20 atoms: what the LDS holds", MM, (150, 450, 700), V, [5, 1, 1, 30, 3, 1, 1, 150, 14, 50, 1], 7),
    ("24 atoms", MM, (120, 90, 700), V, [2, 1, 1, 60, 1, 1, 1, 90, 14, 50, 1], 0),
    ("odd columns, more workgroups than compute units", MM, (300, 465, 501), V, [20, 1, 1, 15, 31, 1, 1, 15, 167, 3, 1], 2),
    ("odd tiles of even rows", BMM, (30, 60, 150, 510), V, [30, 1, 2, 1, 1, 30, 6, 1, 1, 25, 17, 30, 1], 2),
    ("odd rows of a transposed first operand", TA, (30, 75, 160, 502), V, [30, 1, 3, 1, 1, 25, 5, 1, 1, 32, 251, 2, 1], 2),
    ("even columns, more workgroups than compute units", MM, (300, 480, 502), V, [20, 1, 1, 15, 30, 1, 1, 16, 251, 2, 1], 0),
    ("odd columns, 1040 of them", MM, (390, 600, 501), V, [26, 1, 1, 15, 40, 1, 1, 15, 167, 3, 1], 0),
    ("split reduction", MM, (60, 45, 960), K3, [2, 1, 1, 30, 3, 1, 1, 15, 2, 15, 32, 1], 0),
]


def _defs(op, variant, cfg):
    return {m.group(1): int(m.group(2)) for m in re.finditer(r"-D(\w+)=(-?\d+)(?=\s|$)", P.opevo_kernel_defines(op, variant, cfg))}


def _odd16(n):
    return ((n + 15) // 16 | 1) * 16


class Operand:
    """An operand's matrix of one batch, stored [own axis][reduction] (kc) or [reduction][own axis], inside a buffer with nothing behind it."""

    def __init__(self, rng, kc, own, K, tile):
        self.kc, self.own, self.K, self.tile = kc, own, K, tile
        self.mem = rng.permutation(own * K).astype(np.float64)
        self.atoms, self.c = -(-tile // 16), -(-tile // 8)
        self.ld = 40 if kc else _odd16(self.atoms * 16)
        self.part = self.atoms * 16 * self.ld if kc else 32 * self.ld + 192
        self.pieces = tile * 4 if kc else 32 * self.c
        self.odd = K % 2 != 0 if kc else own % 2 != 0 or (tile % 2 != 0 and own > tile)

    def value(self, x, k):
        return self.mem[x * self.K + k] if self.kc else self.mem[k * self.own + x]

    def start(self, x0):
        return min(x0, self.own - 8 * self.c) if not self.kc and self.own >= 8 * self.c else x0

    def step(self, x0, s, nstep):
        """The wave's part of the LDS after step s of the tile at x0 has been stored; NaN where nothing was."""
        S, K = np.full(self.part, np.nan), self.K
        last = s == nstep - 1
        k0 = K - 32 if last else s * 32
        base = x0 * K + k0 if self.kc else k0 * self.own + self.start(x0)
        for q in range(-(-self.pieces // 64) * 64):
            p = q if q < self.pieces else 0                  # a lane without a piece loads the first one and stores nothing
            row, c = divmod(p, 4 if self.kc else self.c)
            g = row * (K if self.kc else self.own) + c * 8
            sh = 0
            if not self.kc and self.own < 8 * self.c and last and q == self.pieces - 1:
                sh = 8 * self.c - self.own
            at = base + g - sh
            odd = at & 1 if self.odd else 0                  # loaded from one element to the left, the last one by itself
            assert self.odd or at % 2 == 0, "a piece that is not 4-byte aligned"
            assert g - sh + (base & 1) >= 0 and at - odd >= 0 and at + 8 <= self.mem.size, (x0, s, q)
            v = np.concatenate([self.mem[at - odd:at - odd + 8], self.mem[at + 7:at + 8]])[odd:odd + 8]
            v = np.concatenate([v[sh:], np.zeros(sh)])
            to = row * self.ld + c * 8 if self.kc else row * self.ld + (row >> 3) * 64 + c * 8
            assert to % 8 == 0 and to + 8 <= self.part
            if q < self.pieces:
                S[to:to + 8] = v
        return S, k0

    def fragments(self, S):
        """What lane l of an atom is given: [atom][lane][8] for positions 8 * (l / 16) on."""
        out = np.empty((self.atoms, 64, 8))
        for a in range(self.atoms):
            for l in range(64):
                if self.kc:
                    at = (a * 16 + l % 16) * self.ld + l // 16 * 8
                    assert at % 8 == 0 and at + 8 <= self.part
                    out[a, l] = S[at:at + 8]
                    continue
                for half in range(2):                        # lane s of a group of 16 addresses 4 elements of row s / 4; lane i receives element i of 4 rows
                    rows = []
                    for r in range(4):
                        k = 8 * (l // 16) + 4 * half + r
                        first = 8 * (l // 16) * self.ld + (8 * (l // 16) >> 3) * 64 + (r + 4 * half) * self.ld + a * 16
                        assert first == k * self.ld + (k >> 3) * 64 + a * 16 and first % 4 == 0 and first + 16 <= self.part
                        rows.append(S[first + l % 16])
                    out[a, l, 4 * half:4 * half + 4] = rows
        return out


@pytest.mark.parametrize("label,kind,dims,variant,cfg,waves", CASES, ids=[c[0] for c in CASES])
def test_which_members_share_it_and_every_address(label, kind, dims, variant, cfg, waves):
    op = P.opevo_op_create(kind, dims, P.OPEVO_BF16)
    plan, D = P.opevo_kernel_plan(op, variant, cfg), _defs(op, variant, cfg)
    assert plan.status == P.OPEVO_OK and plan.path == 6 and D.get("KWAVES", 0) == waves, (plan.path, plan.reason, D.get("KWAVES"))
    if not waves:
        return
    M, N, K, BM, BN = (D[k] for k in "M N K BM BN".split())
    rng, nstep = np.random.default_rng(3), -(-K // 32)
    a, b = Operand(rng, not D["A_TRANS"], M, K, BM), Operand(rng, False, N, K, BN)
    red = a.atoms * 16 * (b.atoms * 16 + 4) * 4
    assert plan.block == 64 * waves <= 1024 and plan.lds_bytes == waves * max(2 * (a.part + b.part), red) <= 160 * 1024
    bounds = [nstep * w // waves for w in range(waves + 1)]
    assert all(y > x for x, y in zip(bounds, bounds[1:])) and bounds[-1] == nstep
    dup = nstep * 32 - K
    for o in (a, b):
        for x0 in {0, o.own - o.tile, (o.own // o.tile - 2) * o.tile if o.own > o.tile else 0}:
            shift = x0 - o.start(x0)
            assert 0 <= shift and shift + o.tile <= o.atoms * 16
            seen = np.zeros(K, int)
            for s in sorted({0, 1, nstep // 2, nstep - 2, nstep - 1} & set(range(nstep))):
                S, k0 = o.step(x0, s, nstep)
                f = o.fragments(S)
                for x in range(o.tile):
                    row = shift + x
                    for g in range(4):
                        got = f[row // 16, row % 16 + 16 * g]
                        for e in range(8):
                            if s < nstep - 1 or 8 * g + e >= dup:    # the last step leaves out what the one before it had
                                assert got[e] == o.value(x0 + x, k0 + 8 * g + e)
                                seen[k0 + 8 * g + e] += x == 0
            assert seen.max() <= 1 and (nstep > 5 or seen.min() == 1)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("label,kind,dims,variant,cfg,waves", [c for c in CASES if c[-1]], ids=[c[0] for c in CASES if c[-1]])
def test_results_match_the_oracle(label, kind, dims, variant, cfg, waves, dtype):
    """Products of 16-bit values are exact in fp32; sums of at most 1310 of them, in 4 parts and more: 5e-6 is 40 roundings."""
    import torch
    from oracle import tensor as T
    make = {MM: synth.matmul_inputs, BMM: synth.bmm_inputs, TA: synth.bmm_ta_inputs}[kind]
    a, b = make(*dims, dtype, 5)
    want = (T.matmul(a, b) if kind == MM else T.bmm(a if kind == BMM else np.ascontiguousarray(a.transpose(0, 2, 1)), b)).ravel()
    op = P.opevo_op_create(kind, dims, synth.DTYPE_CODE[dtype])
    da, db = synth.to_device(a, dtype), synth.to_device(b, dtype)
    dc = torch.full((want.size,), float("nan"), device="cuda:0")
    kernel, _ = P.opevo_kernel_build(op, variant, cfg)
    for _ in range(2):                                       # the second launch overwrites what the first one left
        P.opevo_kernel_launch(kernel, da.data_ptr(), db.data_ptr(), dc.data_ptr(), torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    P.opevo_kernel_destroy(kernel)
    got = dc.cpu().numpy().astype(np.float64)
    assert np.all(np.isfinite(got)) and np.linalg.norm(got - want) <= 5e-6 * np.linalg.norm(want), label


@pytest.mark.gpu
def test_what_lies_beside_a_tile_does_not_reach_it():
    """Infinities and NaN in rows, columns and reduction positions: each shows in its own row or column only, also where the last step repeats positions."""
    import torch
    kind, dims, variant, cfg = MM, (90, 66, 460), V, [3, 1, 1, 30, 3, 1, 1, 22, 46, 10, 1]
    op = P.opevo_op_create(kind, dims, P.OPEVO_BF16)
    assert _defs(op, variant, cfg).get("KWAVES", 0) > 1
    g = torch.Generator().manual_seed(1)
    a, b = torch.randn(90, 460, generator=g).abs() + 0.5, torch.randn(460, 66, generator=g).abs() + 0.5
    a[30, 459], a[59, 430], b[458, 21], b[435, 44] = float("inf"), float("nan"), float("inf"), float("nan")
    a, b = a.to(torch.bfloat16).cuda(), b.to(torch.bfloat16).cuda()
    c = torch.empty(90, 66, device="cuda")
    kernel, _ = P.opevo_kernel_build(op, variant, cfg)
    P.opevo_kernel_launch(kernel, a.data_ptr(), b.data_ptr(), c.data_ptr(), torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    P.opevo_kernel_destroy(kernel)
    want = (a.double().cpu() @ b.double().cpu()).numpy()
    got = c.double().cpu().numpy()
    assert np.array_equal(np.isnan(got), np.isnan(want)) and np.array_equal(np.isinf(got), np.isinf(want))
    fin = np.isfinite(want)
    assert np.linalg.norm(got[fin] - want[fin]) <= 5e-6 * np.linalg.norm(want[fin])
