"""The explicit 128-bit loads of the locked training kernels, held to the rule of
test_asm_discipline.py: nothing touches a load's registers before its wait.  A locked kernel has
three of them: the source row, a sample row under its lock, the source row under its lock."""
import os
import subprocess

import pytest

from paper_2008_12336_amd import build as B
from tests.test_asm_discipline import ROOT, violations


@pytest.mark.timeout(900)
def test_nothing_touches_an_explicit_load_of_a_locked_kernel(tmp_path):
    total_kernels = total_loads = 0
    for unit in ("gosh_train.hip", "gosh_parts.hip"):
        out = str(tmp_path / (unit + ".s"))
        flags = [f for f in B.FLAGS if f not in ("-shared", "-fPIC")]
        subprocess.run([B.hipcc(), *flags, "--cuda-device-only", "-S", "-I" + os.path.join(ROOT, "include"),
                        "-I" + B.CSRC, "-x", "hip", os.path.join(B.CSRC, unit), "-o", out], check=True, capture_output=True)
        text = open(out).read().replace("_ZN4gosh10sgd_kernel", "_ZN4gosh10sgd_unlocked")
        with open(out, "w") as f:
            f.write(text.replace("_ZN4gosh17sgd_locked_kernel", "_ZN4gosh10sgd_kernel"))
        kernels, loads, bad = violations(out)
        assert not bad, "\n".join(bad[:20])
        total_kernels += kernels
        total_loads += loads
    assert total_kernels >= 30 and total_loads >= 3 * total_kernels
