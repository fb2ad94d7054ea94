"""The assembly of the kernels that copy memory to LDS without passing the
registers (load_lds16): such a load reads its LDS address from M0, and gfx950
needs one wait state between the scalar write of M0 and the load (an
instruction in between, or an s_nop).  The compiler inserts none inside an
inline-asm block, and nothing at run time would report a load that took the
previous address.  No GPU needed: hipcc writes the assembly."""
import os
import re
import subprocess

import pytest

from paper_2608_10362_amd import build


def _instructions(src, tmp_path):
    out = str(tmp_path / (src + ".s"))
    flags = [f for f in build.FLAGS if f not in ("-shared", "-fPIC")]
    subprocess.run([build.HIPCC, *flags, "--offload-device-only", "-S", "-I", build.INCLUDE, "-I", build.CSRC,
                    os.path.join(build.CSRC, src), "-o", out], check=True, stdout=subprocess.PIPE,
                   stderr=subprocess.STDOUT, timeout=600)
    lines = (line.split(";")[0].strip() for line in open(out))
    return [line for line in lines if line and not line.startswith(".") and not line.endswith(":")]


@pytest.mark.parametrize("src", ["gemm_tile.hip", "attention.hip"])
def test_m0_settles_before_a_load_to_lds(src, tmp_path):
    ins = _instructions(src, tmp_path)
    loads = [i for i, line in enumerate(ins) if re.match(r"buffer_load_\w+ .*\blds\b", line)]
    assert loads  # (the kernels of this file use the helper)
    close = [ins[i - 1] + " / " + ins[i] for i in loads if re.match(r"s_\w+ m0\b", ins[i - 1])]
    assert not close, f"{len(close)} of {len(loads)} loads directly after M0's write, e.g. {close[0]}"
