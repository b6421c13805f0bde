"""Direct-to-LDS members: gfx9 asks for five wait states between a vector instruction that writes a scalar register and a memory
instruction that reads it as its address.  The template's loads are inline assembly, where the compiler puts none.  The code
objects of members with many scalar registers (bases put aside in vector registers and read back right before the load) are
disassembled and every memory instruction is followed back."""
import glob
import os
import re
import subprocess

import pytest

import paper_2006_05664_amd as P

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
V4, V4A = P.OPEVO_TILE4, P.OPEVO_TILE4A
CASES = [   # kind, dims, space, configuration
    (P.OPEVO_MATMUL, (256, 256, 256), V4, [1, 2, 1, 128, 8, 1, 1, 32, 2, 128, 1]),      # three states before the load
    (P.OPEVO_MATMUL, (256, 256, 256), V4, [1, 1, 2, 128, 8, 1, 1, 32, 8, 32, 1]),
    (P.OPEVO_MATMUL, (8192, 8192, 8192), V4A, [32, 2, 16, 8, 256, 1, 2, 16, 32, 256, 1, 1]),
    (P.OPEVO_BMM, (960, 128, 64, 128), V4, [24, 40, 1, 1, 2, 64, 1, 1, 1, 64, 4, 32, 1]),
    (P.OPEVO_BMM_TA, (960, 128, 64, 128), V4, [320, 3, 1, 1, 8, 16, 2, 1, 16, 2, 4, 32, 1]),
]


def _sregs(text):
    m = re.match(r"s\[(\d+):(\d+)\]$", text)
    if m:
        return set(range(int(m[1]), int(m[2]) + 1))
    m = re.match(r"s(\d+)$", text)
    return {int(m[1])} if m else {"vcc": {106, 107}, "vcc_lo": {106}, "vcc_hi": {107}}.get(text, set())


def short_of_wait_states(asm):
    """Memory instructions that read a scalar register fewer than five states after a vector instruction wrote it."""
    ins = [re.sub(r"//.*|;.*", "", line).split(None, 1) for line in asm.splitlines() if line.startswith("\t")]
    ins = [(p[0], p[1].strip() if len(p) > 1 else "") for p in ins if p]
    short = []
    for i, (op, args) in enumerate(ins):
        if not op.startswith(("global_", "buffer_", "flat_", "scratch_")):
            continue
        need = set().union(*(_sregs(a.strip().split(" ")[0]) for a in args.split(",")))
        states, j = 0, i - 1
        while need and states < 5 and j >= 0:
            o, a = ins[j]
            written = _sregs(a.split(",")[0].strip()) if a else set()
            if o.startswith("v_") and written & need:
                short.append((ins[j], states, ins[i]))
                break
            if o.startswith("s_") and not o.startswith(("s_cmp", "s_bitcmp", "s_nop", "s_waitcnt", "s_barrier", "s_cbranch", "s_branch")):
                need = need - written             # a scalar instruction waits, and its result may be read at once
            states += int(a, 0) + 1 if o == "s_nop" else 1
            j -= 1
    return short


def test_the_check_itself():
    bad = "\tv_readlane_b32 s2, v9, 1\n\tv_readlane_b32 s3, v9, 2\n\ts_mov_b32 m0, s7\n\ts_nop 0\n\tglobal_load_lds_dwordx4 v1, s[2:3]\n"
    assert len(short_of_wait_states(bad)) == 1
    assert not short_of_wait_states(bad.replace("s_nop 0", "s_nop 3"))
    assert not short_of_wait_states(bad.replace("s_nop 0", "s_mov_b64 s[8:9], s[2:3]").replace("v1, s[2:3]", "v1, s[8:9]"))


@pytest.mark.parametrize("kind,dims,variant,cfg", CASES, ids=[str(c[3]) for c in CASES])
def test_no_load_reads_a_scalar_register_too_early(kind, dims, variant, cfg, tmp_path):
    op = P.opevo_op_create(kind, dims, P.OPEVO_BF16)
    assert P.opevo_kernel_plan(op, variant, cfg).path == 3
    P.opevo_code_cache_configure(str(tmp_path), 0)          # the cache's directory: where the code object can be read
    try:
        kernel, _ = P.opevo_kernel_build(op, variant, cfg)
        P.opevo_kernel_destroy(kernel)
    finally:
        P.opevo_code_cache_configure(None, 256 << 20)
    entry = open(glob.glob(os.path.join(str(tmp_path), "*"))[0], "rb").read()
    code = tmp_path / "kernel.co"
    code.write_bytes(entry[entry.index(b"\x7fELF"):])
    asm = subprocess.run([OBJDUMP, "-d", "--mcpu=gfx950", str(code)], capture_output=True, text=True, check=True).stdout
    assert asm.count("global_load_lds_dwordx4") > 8
    assert short_of_wait_states(asm) == []
