"""CPU re-computation of the ragged MFMA template (MatMul / BatchMatMul whose extents are no multiples of 16): every global
load lies inside its operand's matrix, every LDS store and fragment read inside the stage and aligned for its width, and the
fragments hold the operand's values (zeros past the reduction's end) for every row and column of the tile -- for every
tile, thread, piece and slab of small operators (of more than 20 tiles along an axis the first two and the last six: a piece
of 8 reaches past the row's end from no tile further left), with index arithmetic of its own for what is expected."""
import re
import subprocess

import numpy as np
import pytest

import paper_2006_05664_amd as P

CASES = [   # label, kind, dims, space, configuration
    ("125 x 8 tiles, slabs of 100", P.OPEVO_MATMUL, (1000, 1000, 200), P.OPEVO_TILE4, [50, 4, 1, 5, 10, 5, 20, 1, 2, 100, 1]),
    ("every extent odd, rows at odd offsets", P.OPEVO_MATMUL, (27, 35, 45), P.OPEVO_TILE4, [3, 1, 1, 9, 5, 1, 1, 7, 5, 9, 1]),
    ("one tile, one slab, single stage", P.OPEVO_MATMUL, (21, 25, 33), P.OPEVO_TILE4, [1, 1, 1, 21, 1, 1, 1, 25, 1, 33, 0]),
    ("reduction of 8, columns of 8", P.OPEVO_MATMUL, (9, 8, 8), P.OPEVO_TILE4, [1, 1, 1, 9, 1, 1, 1, 8, 1, 8, 1]),
    ("17 columns and one more than 128 steps", P.OPEVO_MATMUL, (40, 34, 129), P.OPEVO_TILE4, [2, 2, 1, 10, 2, 1, 1, 17, 1, 129, 1]),
    ("reduction split over 3 workgroups", P.OPEVO_MATMUL, (36, 55, 105), P.OPEVO_TILE4K, [2, 1, 1, 18, 5, 1, 1, 11, 3, 7, 5, 1]),
    ("launch order", P.OPEVO_MATMUL, (36, 55, 64), P.OPEVO_TILE4X, [2, 1, 1, 18, 5, 1, 1, 11, 2, 32, 1, 1, 0, 2]),
    ("batches, two per workgroup", P.OPEVO_BMM, (6, 20, 27, 50), P.OPEVO_TILE4, [3, 2, 1, 1, 1, 20, 3, 1, 1, 9, 2, 25, 1]),
    ("batches without the lds flag", P.OPEVO_BMM, (3, 33, 40, 48), P.OPEVO_TILE4, [3, 1, 3, 1, 1, 11, 2, 2, 1, 10, 1, 48, 0]),
    ("first operand transposed, odd rows", P.OPEVO_BMM_TA, (4, 27, 33, 70), P.OPEVO_TILE4, [4, 1, 1, 3, 1, 9, 3, 1, 1, 11, 2, 35, 1]),
    ("3 columns: three tiles reach past the row's end", P.OPEVO_MATMUL, (16, 33, 64), P.OPEVO_TILE4, [1, 1, 1, 16, 11, 1, 1, 3, 1, 64, 1]),
    ("3 columns, rows of 9", P.OPEVO_MATMUL, (48, 9, 40), P.OPEVO_TILE4, [1, 1, 1, 48, 3, 1, 1, 3, 2, 20, 1]),
    ("2 columns", P.OPEVO_MATMUL, (16, 34, 64), P.OPEVO_TILE4, [1, 1, 1, 16, 17, 1, 1, 2, 1, 64, 1]),
    ("4 columns", P.OPEVO_MATMUL, (20, 28, 48), P.OPEVO_TILE4, [1, 1, 1, 20, 7, 1, 1, 4, 2, 24, 1]),
    ("5 columns", P.OPEVO_MATMUL, (20, 35, 48), P.OPEVO_TILE4, [1, 1, 1, 20, 7, 1, 1, 5, 2, 24, 1]),
    ("9 columns", P.OPEVO_MATMUL, (20, 27, 48), P.OPEVO_TILE4, [1, 1, 1, 20, 3, 1, 1, 9, 2, 24, 1]),
    ("first operand transposed, 3 rows", P.OPEVO_BMM_TA, (2, 33, 48, 64), P.OPEVO_TILE4, [2, 1, 11, 1, 1, 3, 1, 1, 1, 48, 1, 64, 1]),
    ("first operand transposed, 2 rows", P.OPEVO_BMM_TA, (2, 18, 16, 40), P.OPEVO_TILE4, [1, 2, 9, 1, 1, 2, 1, 1, 1, 16, 2, 20, 1]),
    ("first operand transposed, columns of 8", P.OPEVO_BMM_TA, (2, 8, 24, 100), P.OPEVO_TILE4, [2, 1, 1, 1, 1, 8, 1, 1, 1, 24, 4, 25, 1]),
]


def _defs(op, variant, cfg):
    text = P.opevo_kernel_defines(op, variant, cfg)
    tmpl, rest = text.split(":", 1)
    return tmpl.strip(), {m.group(1): int(m.group(2)) for m in re.finditer(r"-D(\w+)=(-?\d+)(?:\s|$)", rest)}


def _odd16(n):
    return ((n + 15) // 16 | 1) * 16


def _tiles(n):
    return range(n) if n <= 20 else [0, 1] + list(range(n - 6, n))


class Operand:
    """One operand's matrix of a batch as (reduction, own axis), and how the template stages it."""

    def __init__(self, mem, contiguous_k, own_tile, waves, atoms, D):
        self.mem, self.kc, self.tile, self.D = mem, contiguous_k, own_tile, D
        self.rows = waves * atoms * 16
        self.ld = D["KS"] + 8 if contiguous_k else _odd16(self.rows)
        self.stage = self.rows * self.ld if contiguous_k else D["KS"] * self.ld + D["KS"] // 8 * 64

    def off(self, k, x):
        return x * self.ld + k if self.kc else k * self.ld + (k >> 3) * 64 + x

    def fill(self, x0, kb, kpart, k0):
        """The stage after a slab: NaN where nothing was stored."""
        D, KS, flat = self.D, self.D["KS"], self.mem.ravel()
        S = np.full(self.stage, np.nan)
        last = k0 // KS == D["NSL"] - 1
        ck, cx = KS // 8, (self.tile + 7) // 8
        n_pieces = self.tile * ck if self.kc else KS * cx
        for q in range(n_pieces):                 # piece q is thread q % NT's number q / NT
            if self.kc:
                row, c = divmod(q, ck)
                length = self.mem.shape[1]        # K
                k = k0 + c * 8
                start = (x0 + row) * length + kb + min(k, kpart - 8)
                assert kb <= kb + min(k, kpart - 8) and min(k, kpart - 8) + 8 <= kpart
                v = flat[start:start + 8]
                sh = max(k - (kpart - 8), 0) if last else 0
                dst = self.off(c * 8, row)
            else:
                kr, c = divmod(q, cx)
                length = self.mem.shape[1]        # M or N
                k, x = k0 + kr, min(x0 + c * 8, length - 8)
                start = (kb + min(k, kpart - 1)) * length + x
                assert 0 <= x and x + 8 <= length
                v = flat[start:start + 8]
                sh = max(x0 + c * 8 - (length - 8), 0)
                dst = self.off(kr, c * 8)
                if last and k >= kpart:
                    v = np.zeros(8)
            assert start >= 0 and start + 8 <= flat.size and v.size == 8
            v = np.zeros(8) if sh >= 8 else np.concatenate([v[sh:], np.zeros(sh)])
            assert dst % 8 == 0 and dst + 8 <= self.stage
            S[dst:dst + 8] = v
        return S

    def value(self, k, x):
        return self.mem[x, k] if self.kc else self.mem[k, x]

    def check(self, x0, kb, kpart, k0):
        S = self.fill(x0, kb, kpart, k0)
        for x in range(self.rows):
            for k in range(0, self.D["KS"], 8):
                if self.kc:
                    at = self.off(k, x)
                    assert at % 8 == 0 and at + 8 <= self.stage
                    got = S[at:at + 8]
                else:                             # lane s of a group of 16 addresses 4 columns of row k + s / 4
                    for half in (0, 4):
                        at = self.off(k, 0) + half * self.ld + 3 * self.ld + x // 4 * 4
                        assert at % 4 == 0 and at + 4 <= self.stage
                    got = np.array([S[self.off(k, 0) + j * self.ld + x] for j in range(8)])
                if x < self.tile:
                    want = [self.value(kb + k0 + k + j, x0 + x) if k0 + k + j < kpart else 0.0 for j in range(8)]
                    assert np.array_equal(got, want), (x, k, got, want)


def _check_member(kind, dims, variant, cfg):
    op = P.opevo_op_create(kind, dims, P.OPEVO_BF16)
    plan = P.opevo_kernel_plan(op, variant, cfg)
    tmpl, D = _defs(op, variant, cfg)
    assert plan.status == P.OPEVO_OK and plan.path == 6 and tmpl == "gemm_ragged", (plan.path, plan.reason)
    M, N, K, BM, BN = D["M"], D["N"], D["K"], D["BM"], D["BN"]
    kpart = K // D.get("KSPLIT", 1)
    assert plan.block == D["NT"] == 64 * D["WM"] * D["WN"] <= 1024 and D["NSTG"] == (2 if D["NSL"] > 1 and (cfg[-1] != 0 or kind != P.OPEVO_MATMUL) else 1)
    assert plan.grid[0] * plan.grid[1] * plan.grid[2] * BM * BN * D["BATCH_INNER"] == P.opevo_op_sizes(op)[2] * D.get("KSPLIT", 1)
    rng = np.random.default_rng(1)
    a = Operand(rng.random((K, M) if D["A_TRANS"] else (M, K)), not D["A_TRANS"], BM, D["WM"], D["MI"], D)
    b = Operand(rng.random((K, N)), False, BN, D["WN"], D["NI"], D)
    assert D["NSTG"] * (a.stage + b.stage) * 2 == plan.lds_bytes <= 160 * 1024
    for z in range(D.get("KSPLIT", 1)):
        for s in range(D["NSL"]):
            for m in _tiles(M // BM):
                a.check(m * BM, z * kpart, kpart, s * D["KS"])
            for n in _tiles(N // BN):
                b.check(n * BN, z * kpart, kpart, s * D["KS"])


@pytest.mark.parametrize("label,kind,dims,variant,cfg", CASES, ids=[c[0] for c in CASES])
def test_every_address_and_every_fragment_value(label, kind, dims, variant, cfg):
    _check_member(kind, dims, variant, cfg)
    op = P.opevo_op_create(kind, dims, P.OPEVO_BF16)
    kernel, _ = P.opevo_kernel_build(op, variant, cfg)
    assert 1000 < P.opevo_kernel_code_size(kernel) < (128 << 10)
    P.opevo_kernel_destroy(kernel)


@pytest.mark.parametrize("kind,dims", [(P.OPEVO_MATMUL, (20, 33, 45)), (P.OPEVO_MATMUL, (48, 18, 30)), (P.OPEVO_BMM, (2, 30, 50, 20)),
                                       (P.OPEVO_BMM_TA, (2, 18, 27, 40))])
def test_every_address_and_every_fragment_value_of_random_members(kind, dims):
    op = P.opevo_op_create(kind, dims, P.OPEVO_BF16)
    sp, rng, found = P.opevo_op_space(op, P.OPEVO_TILE4), P.opevo_rng_create(3), []
    while len(found) < 15:
        cfg = P.opevo_space_random(sp, rng)
        if P.opevo_kernel_plan(op, P.OPEVO_TILE4, cfg).path == 6:
            found.append([int(x) for x in cfg])
    for cfg in found:
        _check_member(kind, dims, P.OPEVO_TILE4, cfg)
    P.opevo_rng_destroy(rng); P.opevo_space_destroy(sp)


MANY_ATOMS = [   # members whose tile fits nine waves better than eight, where a lane has 170 registers instead of 256
    ("20 atom columns", P.OPEVO_MATMUL, (231, 945, 330), P.OPEVO_TILE4, [7, 1, 11, 3, 1, 9, 21, 5, 330, 1, 1]),
    ("9 x 14 atoms", P.OPEVO_MATMUL, (360, 840, 600), P.OPEVO_TILE4, [9, 10, 2, 2, 1, 60, 14, 1, 20, 30, 1]),
    ("first operand transposed, 23 x 7 atoms", P.OPEVO_BMM_TA, (8, 360, 420, 250), P.OPEVO_TILE4, [4, 2, 1, 120, 3, 1, 3, 5, 7, 4, 250, 1, 1]),
    ("first operand transposed, one stage", P.OPEVO_BMM_TA, (8, 360, 420, 250), P.OPEVO_TILE4, [1, 8, 4, 5, 9, 2, 1, 35, 3, 4, 125, 2, 0]),
]


@pytest.mark.parametrize("label,kind,dims,variant,cfg", MANY_ATOMS, ids=[c[0] for c in MANY_ATOMS])
def test_the_division_among_waves_leaves_registers_enough(label, kind, dims, variant, cfg, tmp_path):
    """A kernel with scratch memory (spilled registers) is refused at its first launch."""
    op = P.opevo_op_create(kind, dims, P.OPEVO_BF16)
    assert P.opevo_kernel_plan(op, variant, cfg).path == 6
    P.opevo_code_cache_configure(str(tmp_path), 0)          # the cache's directory: where the code object can be read
    try:
        kernel, _ = P.opevo_kernel_build(op, variant, cfg)
        P.opevo_kernel_destroy(kernel)
    finally:
        P.opevo_code_cache_configure(None, 256 << 20)
    entry = next(tmp_path.iterdir()).read_bytes()
    code = tmp_path / "kernel.co"
    code.write_bytes(entry[entry.index(b"\x7fELF"):])
    notes = subprocess.run(["/opt/rocm/llvm/bin/llvm-readelf", "--notes", str(code)], capture_output=True, text=True, check=True).stdout
    assert re.search(r"private_segment_fixed_size:\s+0\b", notes), re.findall(r"private_segment_fixed_size:\s+\d+", notes)


def test_which_members_take_the_ragged_template():
    def path(kind, dims, variant, cfg, dtype=P.OPEVO_BF16):
        plan = P.opevo_kernel_plan(P.opevo_op_create(kind, dims, dtype), variant, cfg)
        assert plan.status == P.OPEVO_OK
        return plan.path
    V = P.OPEVO_TILE4
    assert path(P.OPEVO_MATMUL, (36, 55, 64), V, [2, 1, 1, 18, 5, 1, 1, 11, 2, 32, 1]) == 6
    assert path(P.OPEVO_MATMUL, (36, 55, 64), V, [2, 1, 1, 18, 5, 1, 1, 11, 2, 32, 1], P.OPEVO_F32) == 0    # 16-bit inputs only
    assert path(P.OPEVO_MATMUL, (48, 80, 64), V, [6, 1, 1, 8, 10, 1, 1, 8, 2, 32, 1]) == 0      # extents of whole atoms: the member asked for the scalar tile
    assert path(P.OPEVO_MATMUL, (36, 55, 64), V, [36, 1, 1, 1, 5, 1, 1, 11, 2, 32, 1]) == 0     # a single row: 23 times the work
    assert path(P.OPEVO_MATMUL, (36, 7, 64), V, [2, 1, 1, 18, 1, 1, 1, 7, 2, 32, 1]) == 0       # rows shorter than a piece
    assert path(P.OPEVO_MATMUL, (36, 55, 7), V, [2, 1, 1, 18, 5, 1, 1, 11, 1, 7, 1]) == 0
    assert path(P.OPEVO_MATMUL, (1000, 1000, 1000), V, [1, 25, 5, 8, 10, 100, 1, 1, 200, 5, 0]) == 0     # 441 atoms: too many for eight waves
    assert path(P.OPEVO_MATMUL, (36, 55, 64), P.OPEVO_TILE2, [2, 18, 5, 11, 2, 32]) == 0


def test_random_members_of_ragged_operators_reach_the_template():
    """Every member on the ragged template is valid and within the limits, and a share of a ragged space is on it."""
    for kind, dims in ((P.OPEVO_MATMUL, (1000, 1000, 1000)), (P.OPEVO_MATMUL, (231, 945, 330)), (P.OPEVO_BMM, (30, 60, 105, 50)),
                       (P.OPEVO_BMM_TA, (30, 60, 105, 50))):
        op = P.opevo_op_create(kind, dims, P.OPEVO_BF16)
        sp, rng = P.opevo_op_space(op, P.OPEVO_TILE4), P.opevo_rng_create(3)
        n = {}
        for _ in range(600):
            cfg = P.opevo_space_random(sp, rng)
            plan = P.opevo_kernel_plan(op, P.OPEVO_TILE4, cfg)
            n[plan.path] = n.get(plan.path, 0) + 1
            if plan.path == 6:
                assert plan.status == P.OPEVO_OK and plan.lds_bytes <= 160 * 1024 and plan.block <= 1024 and plan.acc_per_lane <= 128
        assert n.get(6, 0) > 60, (dims, n)
        P.opevo_rng_destroy(rng); P.opevo_space_destroy(sp)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("label,kind,dims,variant,cfg", CASES + MANY_ATOMS, ids=[c[0] for c in CASES + MANY_ATOMS])
def test_results_match_the_oracle(label, kind, dims, variant, cfg, dtype):
    """Inputs are exact in both precisions; what is left is an fp32 sum of at most 600 products: 1e-5 is 80 roundings."""
    import torch
    from oracle import tensor as T
    from paper_2006_05664_amd import synth
    make = {P.OPEVO_MATMUL: synth.matmul_inputs, P.OPEVO_BMM: synth.bmm_inputs, P.OPEVO_BMM_TA: synth.bmm_ta_inputs}[kind]
    a, b = make(*dims, dtype, 5)
    want = T.matmul(a, b) if kind == P.OPEVO_MATMUL else T.bmm(a if kind == P.OPEVO_BMM else np.ascontiguousarray(a.transpose(0, 2, 1)), b)
    op = P.opevo_op_create(kind, dims, synth.DTYPE_CODE[dtype])
    da, db = synth.to_device(a, dtype), synth.to_device(b, dtype)
    dc = torch.full((want.size,), float("nan"), device="cuda:0")
    kernel, _ = P.opevo_kernel_build(op, variant, cfg)
    for _ in range(2):        # the second launch writes over the first one's output
        P.opevo_kernel_launch(kernel, da.data_ptr(), db.data_ptr(), dc.data_ptr(), torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    P.opevo_kernel_destroy(kernel)
    got = dc.cpu().numpy().astype(np.float64)
    assert np.all(np.isfinite(got))
    assert np.linalg.norm(got - want.ravel()) <= 1e-5 * np.linalg.norm(want), label
