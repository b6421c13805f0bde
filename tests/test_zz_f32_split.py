"""The template that multiplies fp32 values as three bf16 parts each: which members it takes, and its results where its parts meet: every tile, parts of the
reduction of unequal length, four and eight waves, a transposed first operand, batches, values that cannot be taken apart, sums beyond the range."""
import re
import subprocess

import numpy as np
import pytest

import paper_2006_05664_amd as P
from paper_2006_05664_amd import synth
from test_zz_load_base_wait import OBJDUMP, short_of_wait_states

MM, BMM, TA = P.OPEVO_MATMUL, P.OPEVO_BMM, P.OPEVO_BMM_TA
V, X, K3 = P.OPEVO_TILE4, P.OPEVO_TILE4X, P.OPEVO_TILE4K
CASES = [   # label, kind, dims, variant, configuration, waves that share the reduction (0: not on this template)
    ("64 x 64, 29 chunks on four waves", MM, (1024, 1088, 928), V, [16, 2, 1, 32, 17, 2, 1, 32, 29, 32, 1], 4),
    ("32 x 64, 11 chunks on four waves", MM, (64, 128, 352), V, [2, 1, 1, 32, 2, 1, 2, 32, 11, 32, 1], 4),
    ("64 x 32, the shortest reduction", MM, (64, 96, 320), V, [1, 1, 2, 32, 3, 1, 1, 32, 10, 32, 1], 4),
    ("32 x 32, 23 chunks on eight waves", MM, (96, 64, 736), V, [3, 1, 1, 32, 2, 1, 1, 32, 23, 32, 1], 8),
    ("64 x 64, eight waves", MM, (64, 64, 1024), V, [1, 2, 1, 32, 1, 2, 1, 32, 16, 64, 1], 8),
    ("slabs of 8, a launch order of its own", MM, (128, 64, 928), X, [2, 1, 2, 32, 1, 2, 1, 32, 116, 8, 1, 1, 0, 2], 8),
    ("batches, two per workgroup", BMM, (6, 64, 32, 416), V, [3, 2, 2, 1, 1, 32, 1, 1, 1, 32, 13, 32, 1], 4),
    ("transposed first operand, 64 x 32", TA, (4, 64, 96, 448), V, [2, 2, 1, 2, 1, 32, 3, 1, 1, 32, 14, 32, 1], 4),
    ("transposed first operand, 32 x 64", TA, (4, 96, 128, 704), V, [2, 2, 3, 1, 1, 32, 2, 2, 1, 32, 22, 32, 1], 8),
    ("transposed first operand, 32 x 32", TA, (2, 96, 32, 768), V, [2, 1, 3, 1, 1, 32, 1, 1, 1, 32, 24, 32, 1], 8),
    ("64 x 64, workgroups enough for the chip", MM, (1472, 1472, 768), V, [23, 2, 1, 32, 23, 2, 1, 32, 12, 64, 1], 4),
    ("64 x 64, no more of them, shorter", MM, (1024, 2048, 864), V, [16, 2, 1, 32, 32, 2, 1, 32, 27, 32, 1], 0),
    ("64 x 64, workgroups enough, shorter", MM, (1472, 1472, 736), V, [23, 2, 1, 32, 23, 2, 1, 32, 23, 32, 1], 0),
    ("32 x 64, workgroups enough for the chip", MM, (736, 1472, 1056), V, [23, 1, 1, 32, 23, 2, 1, 32, 33, 32, 1], 4),
    ("32 x 64, workgroups enough, shorter", MM, (736, 1472, 1024), V, [23, 1, 1, 32, 23, 2, 1, 32, 16, 64, 1], 0),
    ("64 x 32, no more of them", MM, (1024, 1024, 320), V, [16, 2, 1, 32, 32, 1, 1, 32, 10, 32, 1], 4),
    ("batches on more workgroups", BMM, (401, 32, 32, 1056), V, [401, 1, 1, 1, 1, 32, 1, 1, 1, 32, 33, 32, 1], 0),
    ("transposed first operand, 64 x 64", TA, (4, 64, 128, 1024), V, [2, 2, 1, 2, 1, 32, 2, 2, 1, 32, 32, 32, 1], 0),
    ("32 x 64, shorter", MM, (64, 128, 288), V, [2, 1, 1, 32, 2, 1, 2, 32, 9, 32, 1], 0),
    ("no whole chunks", MM, (64, 128, 336), V, [2, 1, 1, 32, 2, 1, 2, 32, 21, 16, 1], 0),
    ("96 columns", MM, (64, 96, 512), V, [2, 1, 1, 32, 1, 1, 3, 32, 16, 32, 1], 0),
    ("no pipelining asked for", MM, (64, 128, 512), V, [2, 1, 1, 32, 2, 1, 2, 32, 16, 32, 0], 0),
    ("split reduction", MM, (64, 128, 1024), K3, [2, 1, 1, 32, 2, 1, 2, 32, 2, 16, 32, 1], 0),
]


def _waves(kind, dims, variant, cfg):
    op = P.opevo_op_create(kind, dims, P.OPEVO_F32)
    plan = P.opevo_kernel_plan(op, variant, cfg)
    assert plan.status == P.OPEVO_OK and plan.path == 4, (plan.path, plan.reason)
    words = P.opevo_kernel_defines(op, variant, cfg).split()
    return plan.block // 64 if words[0] == "gemm_f32_split:" else 0


@pytest.mark.parametrize("label,kind,dims,variant,cfg,waves", CASES, ids=[c[0] for c in CASES])
def test_which_members_it_takes(label, kind, dims, variant, cfg, waves):
    assert _waves(kind, dims, variant, cfg) == waves


@pytest.mark.parametrize("bm", [32, 64])
def test_where_the_first_operand_s_pieces_go(bm):
    """A chunk of 32 reduction steps, 16 bytes a lane and load: every value once, inside the half it is meant for, where the fragments are read, and the
    16 lanes of a turn of a fragment read on 16 groups of 4 banks."""
    K, lane = 96, np.arange(64)
    lds = np.full(bm * 32, -1)
    a_off = lane // 8 * K + (lane % 8 ^ lane >> 4) * 4                # elements
    for i in range(bm // 8):
        at = a_off ^ 16 if i & 1 else a_off
        for e in range(4):
            assert (lds[i * 256 + lane * 4 + e] == -1).all()
            lds[i * 256 + lane * 4 + e] = i * 8 * K + at + e
    for i in range(bm // 32):
        for t in range(2):
            row, p = i * 32 + lane % 32, 4 * t + 2 * (lane // 32)
            key = row >> 1 & 7
            for half in range(2):
                piece = row * 8 + (p + half ^ key)
                for e in range(4):
                    assert (lds[piece * 4 + e] == row * K + t * 16 + 8 * (lane // 32) + 4 * half + e).all()
                assert all(len(set(piece[g:g + 16] % 16)) == 16 for g in range(0, 64, 16))


@pytest.mark.parametrize("dims,cfg,atoms", [
    ((1024, 1088, 928), [16, 2, 1, 32, 17, 2, 1, 32, 29, 32, 1], (2, 2)),
    ((64, 128, 352), [2, 1, 1, 32, 2, 1, 2, 32, 11, 32, 1], (1, 2)),
    ((64, 96, 320), [1, 1, 2, 32, 3, 1, 1, 32, 10, 32, 1], (2, 1)),
    ((96, 64, 736), [3, 1, 1, 32, 2, 1, 1, 32, 23, 32, 1], (1, 1)),
])
def test_every_fragment_is_read_after_its_loads(dims, cfg, atoms, tmp_path):
    """The loop of the compiled kernel, three times round.  The first operand's loads go to the LDS unseen by the compiler, so the kernel waits for them itself:
    when the fragments of a chunk's second step are read, the chunk's loads were issued two rounds before, when the next chunk's first step is, one round
    before.  Waits leave the youngest loads under way; loads are served in order."""
    op = P.opevo_op_create(MM, dims, P.OPEVO_F32)
    P.opevo_code_cache_configure(str(tmp_path), 0)
    try:
        kernel, _ = P.opevo_kernel_build(op, V, cfg)
        P.opevo_kernel_destroy(kernel)
    finally:
        P.opevo_code_cache_configure(None, 256 << 20)
    files = list(tmp_path.iterdir())
    assert len(files) == 1, "one compilation: it does not spill"
    data = files[0].read_bytes()
    code = tmp_path / "kernel.co"
    code.write_bytes(data[data.index(b"\x7fELF"):])
    asm = subprocess.run([OBJDUMP, "-d", "--mcpu=gfx950", str(code)], capture_output=True, text=True, check=True).stdout
    assert short_of_wait_states(asm) == []
    ins = []                                                  # (address, text)
    for line in asm.splitlines():
        m = re.match(r"\t(.*?)\s*// ([0-9A-F]{12}):", line)
        if m:
            ins.append((int(m[2], 16), m[1].strip()))
    at = {a: i for i, (a, _) in enumerate(ins)}
    loops = []
    for i, (a, t) in enumerate(ins):
        m = re.match(r"s_cbranch_\w+ (\d+)", t)
        if m and int(m[1]) > 32767 and a + 4 + 4 * (int(m[1]) - 65536) in at:
            loops.append([t for _, t in ins[at[a + 4 + 4 * (int(m[1]) - 65536)]:i]])
    body = [b for b in loops if sum("mfma_f32_32x32x16_bf16" in t for t in b) == 16 * atoms[0] * atoms[1]]
    assert len(body) == 1
    body, pieces = body[0], 4 * atoms[0]
    assert sum(t.startswith("global_load_lds") for t in body) == pieces and sum(t.startswith("ds_read_b128") for t in body) == 4 * atoms[0]
    pending = []                                              # rounds of the loads to the LDS under way, None for loads to registers; the oldest first
    for r in range(4):
        reads = 0
        for t in body:
            if t.startswith("global_load_lds"):
                pending.append(r)
            elif t.startswith("global_load"):
                pending.append(None)
            elif t.startswith("s_waitcnt") and "vmcnt" in t:
                left = int(re.search(r"vmcnt\((\d+)\)", t)[1])
                pending = pending[len(pending) - left:] if left < len(pending) else pending
            elif t.startswith("ds_read_b128"):
                done_by = r - 2 if reads < 2 * atoms[0] else r - 1
                assert all(p is None or p > done_by for p in pending), (r, reads, pending)
                reads += 1
            assert not t.startswith(("ds_write", "s_barrier"))


def test_members_that_could_not_run_without_it_stay_invalid():
    """One wave on slabs of 144 would stage 288 registers a lane on the fp32 atoms' template."""
    op = P.opevo_op_create(MM, (64, 64, 1152), P.OPEVO_F32)
    assert P.opevo_kernel_plan(op, V, [1, 1, 2, 32, 1, 1, 2, 32, 8, 144, 1]).status == P.OPEVO_E_INVALID
    assert _waves(MM, (64, 64, 1152), V, [1, 2, 1, 32, 1, 1, 2, 32, 8, 144, 1]) == 8


def _run(kind, dims, variant, cfg, a, b, n):
    import torch
    op = P.opevo_op_create(kind, dims, P.OPEVO_F32)
    da, db = torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0"), torch.from_numpy(np.ascontiguousarray(b)).to("cuda:0")
    dc = torch.full((n,), float("nan"), device="cuda:0")
    kernel, _ = P.opevo_kernel_build(op, variant, cfg)
    for _ in range(2):                                     # the second launch overwrites what the first one left
        P.opevo_kernel_launch(kernel, da.data_ptr(), db.data_ptr(), dc.data_ptr(), torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    P.opevo_kernel_destroy(kernel)
    return dc.cpu().numpy()


@pytest.mark.gpu
@pytest.mark.parametrize("label,kind,dims,variant,cfg,waves", [c for c in CASES if c[-1]], ids=[c[0] for c in CASES if c[-1]])
def test_results_match_the_oracle(label, kind, dims, variant, cfg, waves):
    """A wave adds at most 256 products, 16 at a time: 16 roundings of a growing sum, some 4 of the result's norm by their random signs; the final
    sum has at most 8.  1.2e-6 is 20."""
    from oracle import tensor as T
    a, b = {MM: synth.matmul_inputs, BMM: synth.bmm_inputs, TA: synth.bmm_ta_inputs}[kind](*dims, "f32", 5)
    want = (T.matmul(a, b) if kind == MM else T.bmm(a if kind == BMM else np.ascontiguousarray(a.transpose(0, 2, 1)), b)).ravel()
    got = _run(kind, dims, variant, cfg, a, b, want.size).astype(np.float64)
    assert np.all(np.isfinite(got)) and np.linalg.norm(got - want) <= 1.2e-6 * np.linalg.norm(want), label


FOUR, EIGHT = (MM, (64, 64, 480), V, [1, 2, 1, 32, 2, 1, 1, 32, 15, 32, 1]), (MM, (64, 64, 960), V, [1, 2, 1, 32, 1, 2, 1, 32, 30, 32, 1])
MEMBERS = pytest.mark.parametrize("member", [FOUR, EIGHT], ids=["64 x 32, four waves", "64 x 64, eight waves"])


def test_the_members_of_the_tests_below():
    assert _waves(*FOUR) == 4 and _waves(*EIGHT) == 8


def _operands(member):
    g, K = np.random.default_rng(7), member[1][2]
    return g.standard_normal((64, K)).astype(np.float32), g.standard_normal((K, 64)).astype(np.float32)


@pytest.mark.gpu
@MEMBERS
@pytest.mark.parametrize("scale_a,scale_b", [(2.0 ** -60, 2.0 ** -60), (2.0 ** -99, 2.0 ** 99), (2.0 ** -120, 2.0 ** 100), (2.0 ** -135, 2.0 ** 40), (2.0 ** 118, 1.0)])
def test_operands_of_any_magnitude(member, scale_a, scale_b):
    """Scaling by powers of two changes no relative error as long as the values keep their 24 bits (rounded to fp32 here, as the operands are)."""
    a, b = _operands(member)
    a, b = (a * np.float32(scale_a)).astype(np.float32), (b * np.float32(scale_b)).astype(np.float32)
    want = a.astype(np.float64) @ b.astype(np.float64)
    got = _run(*member, a, b, want.size).astype(np.float64).reshape(want.shape)
    assert np.linalg.norm(got - want) <= 1.2e-6 * np.linalg.norm(want)


@pytest.mark.gpu
@pytest.mark.parametrize("label,kind,dims,variant,cfg,waves", [c for c in CASES if c[-1] and c[1] == MM and c[3] == V], ids=[c[0] for c in CASES if c[-1] and c[1] == MM and c[3] == V])
def test_no_further_from_64_bits_than_the_fp32_atoms(label, kind, dims, variant, cfg, waves):
    """The same operands through the same tile without pipelining, which runs on the fp32 atoms: its sums are rounded eight times for 16 products."""
    a, b = synth.matmul_inputs(*dims, "f32", 5)
    want = a.astype(np.float64) @ b.astype(np.float64)
    off = [np.linalg.norm(_run(kind, dims, variant, cfg[:-1] + [flag], a, b, want.size).reshape(want.shape) - want) for flag in (1, 0)]
    assert _waves(kind, dims, variant, cfg[:-1] + [0]) == 0 and off[0] <= off[1], off


@pytest.mark.gpu
@MEMBERS
@pytest.mark.parametrize("seed", [1, 2])
def test_sums_of_a_single_product(member, seed):
    """Selections and sparse rows: the product of the upper parts is exact, the seven others are at most 2^-7 of it and lose no more than 2^-24 of that
    each time they are added to, so the one rounding of their sum is all but fp32's (2^-24): 2^-24 + 2^-28, and 2 % in the norm."""
    g = np.random.default_rng(seed)
    K = member[1][2]
    a, b = np.zeros((64, K), np.float32), g.standard_normal((K, 64)).astype(np.float32)
    k = g.permutation(K)[:64]
    a[np.arange(64), k] = g.standard_normal(64).astype(np.float32)
    a[0, k[0]] = 1.0
    want = a.astype(np.float64) @ b.astype(np.float64)
    got = _run(*member, a, b, want.size).astype(np.float64).reshape(want.shape)
    rounded = want.astype(np.float32)
    assert np.array_equal(got[0], b[k[0]].astype(np.float64)), "a value times one is that value"
    assert np.all(np.abs(got - want) <= (2.0 ** -24 + 2.0 ** -28) * np.abs(want))
    assert np.linalg.norm(got - want) <= 1.02 * np.linalg.norm(rounded - want)


@pytest.mark.gpu
@MEMBERS
@pytest.mark.parametrize("terms", [2, 3, 4, 8])
def test_sums_of_a_few_products(member, terms):
    """Beside the fp32 atoms of the same tile, which round once for each product: the sums of the upper parts' products (16 bits each) are exact or nearly, those of the
    others 2^-7 of them, so a sum is rounded about once, wherever in the reduction and in whichever waves' parts its products lie.  64 x 64 x 6 sums: their norms
    agree to 1 %, 2 % are allowed."""
    kind, dims, variant, cfg = member
    K, off = dims[2], {0: 0.0, 1: 0.0}
    for seed in range(6):
        g = np.random.default_rng(seed)
        a, b = np.zeros((64, K), np.float32), g.standard_normal((K, 64)).astype(np.float32)
        for i in range(64):
            a[i, g.permutation(K)[:terms]] = g.standard_normal(terms).astype(np.float32)
        want = a.astype(np.float64) @ b.astype(np.float64)
        for flag in off:
            off[flag] += np.linalg.norm(_run(kind, dims, variant, cfg[:-1] + [flag], a, b, want.size).reshape(want.shape) - want) ** 2
    assert _waves(kind, dims, variant, cfg[:-1] + [0]) == 0 and off[1] <= 1.02 ** 2 * off[0], off


@pytest.mark.gpu
@MEMBERS
@pytest.mark.parametrize("scale", [2.0 ** -60, 2.0 ** -64, 2.0 ** -70])
def test_products_that_are_subnormal_or_nearly(member, scale):
    """One product for each output, of values that can be taken apart, whose smaller parts have no 24 bits left: rounded once, as on the fp32 atoms."""
    g = np.random.default_rng(4)
    K = member[1][2]
    a, b = np.zeros((64, K), np.float32), (g.standard_normal((K, 64)) * scale).astype(np.float32)
    a[np.arange(64), g.permutation(K)[:64]] = (g.standard_normal(64) * scale).astype(np.float32)
    assert np.all(np.abs(b) > 2.0 ** -100) and np.all((np.abs(a) > 2.0 ** -100) | (a == 0))
    want = a.astype(np.float64) @ b.astype(np.float64)
    got = _run(*member, a, b, want.size).reshape(want.shape)
    assert np.array_equal(got, want.astype(np.float32))


@pytest.mark.gpu
@MEMBERS
def test_a_single_value_that_cannot_be_taken_apart(member):
    """Rows and columns whose only values lie below 2^-100, one for each place of a lane's 8 and each wave, beside ordinary ones and zeros."""
    a, b = _operands(member)
    K = member[1][2]
    a[np.abs(a) < 0.5] = 0.0
    for i in range(32):
        a[i] = 0.0
        a[i, (i * 37) % K] = np.float32(1.2345678e-34)
        b[:, i] = 0.0
        b[(i * 41) % K, i] = np.float32(-7.654321e-33)
    b[:, 32:] *= np.float32(1e20)
    a[32:] *= np.float32(1e15)
    want = a.astype(np.float64) @ b.astype(np.float64)
    got = _run(*member, a, b, want.size).astype(np.float64).reshape(want.shape)
    for part in (np.s_[:32, 32:], np.s_[32:, :32]):            # one product each: rounded once (2^-24), or a chain of zeros and one product
        assert np.all(np.abs(got[part] - want[part]) <= 2.0 ** -23 * np.abs(want[part]))
    assert np.linalg.norm(got[32:, 32:] - want[32:, 32:]) <= 1.2e-6 * np.linalg.norm(want[32:, 32:])


def _parts(v):
    """A value's three bf16 parts, as the kernel takes it apart: each the rest rounded to nearest, ties to even."""
    out = []
    for _ in range(3):
        u = v.view(np.uint32)
        h = ((u + 0x7fff + (u >> 16 & 1)) & np.uint32(0xffff0000)).view(np.float32)
        out.append(h)
        v = v - h
    return out


def test_which_values_are_no_sum_of_three_parts():
    """Whatever is not the sum of its parts is taken for too small by the kernel's test on its bits; nothing from 2^-100 on is, nor is zero."""
    g = np.random.default_rng(3)
    exps = np.arange(-149, 120)
    v = np.concatenate([(g.uniform(1, 2, (64, 1)) * 2.0 ** exps).astype(np.float32).ravel(), (2.0 ** exps).astype(np.float32), np.zeros(2, np.float32)])
    v = np.concatenate([v, -v])
    small = ((v.view(np.uint32).astype(np.uint64) << 1) - 1 & 0xffffffff) < 2 * (27 << 23) - 1
    assert not small[(np.abs(v) >= 2.0 ** -100) | (v == 0)].any()
    assert small[(np.abs(v) < 2.0 ** -100) & (v != 0)].all()
    assert np.all((sum(p.astype(np.float64) for p in _parts(v)) == v)[~small])
    gone = (_parts(v)[0] == 0) & (v != 0)                      # up to 2^-134 no part has anything of them
    assert gone.any() and small[gone].all() and np.all(np.abs(v[gone]) <= 2.0 ** -134)


@pytest.mark.gpu
@MEMBERS
@pytest.mark.parametrize("scale_a,scale_b", [(2.0 ** -140, 2.0 ** 40), (2.0 ** -140, 2.0 ** 100), (2.0 ** 100, 2.0 ** -138)])
def test_an_operand_wholly_below_what_bf16_holds(member, scale_a, scale_b):
    """Every value at most 2^-134, few bits each: no product has more than 24 + 15, and the sums are the fp32 atoms' (1.2e-6: at most 960 products, as above)."""
    a, b = _operands(member)
    a, b = (np.clip(a, -2, 2) * np.float32(scale_a)).astype(np.float32), (np.clip(b, -2, 2) * np.float32(scale_b)).astype(np.float32)
    tiny = a if scale_a < 1 else b
    assert np.all(np.abs(tiny) <= 2.0 ** -134) and np.mean(tiny != 0) > 0.9
    want = a.astype(np.float64) @ b.astype(np.float64)
    got = _run(*member, a, b, want.size).astype(np.float64).reshape(want.shape)
    assert np.linalg.norm(got - want) <= 1.2e-6 * np.linalg.norm(want)


@pytest.mark.gpu
@MEMBERS
@pytest.mark.parametrize("value", [2.0 ** -149, 2.0 ** -134, 1.5 * 2.0 ** -135])
def test_the_only_value_of_a_wave_s_part(member, value):
    """One product for each row, in the first wave's part, the last one's and one between: exact (the other factor is a power of two)."""
    K = member[1][2]
    a, b = np.zeros((64, K), np.float32), np.zeros((K, 64), np.float32)
    for i, k in enumerate((0, 127, K // 2 - 40, K - 1)):
        a[16 * i + 3, k] = np.float32(value)
        b[k] = np.float32(2.0 ** (100 + i))
    want = a.astype(np.float64) @ b.astype(np.float64)
    got = _run(*member, a, b, want.size).reshape(want.shape)
    assert np.count_nonzero(want) == 4 * 64 and np.array_equal(got.astype(np.float64), want)


@pytest.mark.gpu
@MEMBERS
def test_infinities_nan_and_sums_beyond_the_range(member):
    K = member[1][2]
    a, b = _operands(member)
    a[3, 100], a[4, 101], b[K - 10, 9] = np.inf, np.nan, -np.inf
    a[5], a[6] = 0.0, np.abs(a[6]) * np.float32(2.0 ** 125)    # row 6: every sum of like signs is far beyond the range
    with np.errstate(invalid="ignore"):
        want = a.astype(np.float64) @ np.abs(b).astype(np.float64)
    got = _run(*member, a, np.abs(b), want.size).reshape(want.shape)
    with np.errstate(over="ignore"):
        assert np.array_equal(np.isnan(got), np.isnan(want)) and np.array_equal(np.isinf(got), np.isinf(want.astype(np.float32)))
    # the early products alone leave the range upwards, the late ones downwards, all together upwards: infinite in order, a NaN as the sum of partial sums
    a, b = _operands(member)
    a, b = np.abs(a) * np.float32(2.0 ** 124), np.abs(b)
    b[K // 2:] *= np.float32(-0.25)
    want = a.astype(np.float64) @ b.astype(np.float64)
    got = _run(*member, a, b, want.size).reshape(want.shape)
    assert np.all(np.isfinite(a)) and np.all(want > 3.5e38) and np.all(np.isposinf(got))
