"""What the compiler made of hand-written assembly, read from the listing of a kernel file of this repository (CPU only)."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2502_19078_amd import build


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="no hipcc")
def test_a_load_into_lds_has_a_base_that_no_vector_instruction_wrote(tmp_path):
    """A scalar register that a vector instruction has written may be a load's base five wait states later at the earliest, which nothing checks
    inside assembly: every such load of the stack kernels reads a copy that a scalar instruction made right before it, and m0 is never
    written by a vector instruction."""
    out = str(tmp_path / "stack.s")
    flags = [f for f in build.FLAGS if f not in ("-shared", "-Wall")]
    subprocess.run(["hipcc", *flags, "-I", os.path.join(build.ROOT, "include"), "-I", build.CSRC, "--offload-device-only", "-S",
                    os.path.join(build.CSRC, "ffn_stack.hip"), "-o", out], check=True, capture_output=True, text=True)
    code = [s for s in (line.split(";")[0].strip() for line in open(out)) if s and not s.startswith((".", ";"))]
    loads = 0
    for before, line in zip(code, code[1:]):
        m = re.match(r"global_load_lds_dwordx4 v\d+, (s\[\d+:\d+\])", line)
        if m:
            loads += 1
            assert before.startswith(f"s_mov_b64 {m[1]},"), (before, line)
    assert loads > 500
    assert not [s for s in code if re.match(r"v_\w+ m0\b", s)]
