"""What a ragged MFMA member that is built without kept places asks the compiler for."""
import os
import re
import subprocess

import pytest

import paper_2006_05664_amd as P
from host_code import CLANG, ROOT

V = P.OPEVO_TILE4


def _defs(op, cfg):
    text = P.opevo_kernel_defines(op, V, cfg)
    return text, {m.group(1): int(m.group(2)) for m in re.finditer(r"-D(\w+)=(-?\d+)(?=\s|$)", text)}


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
