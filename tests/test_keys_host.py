"""The slot-table pass's list of up to four keys in registers (tlmpm_keys.h) on the CPU.

tests/native/keys_check.hip is built with hipcc as a host program and goes through every
sequence of eight additions: four distinct codes around a node must stay in registers,
whatever absent entries follow them.
"""
import os
import re
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.mark.skipif(shutil.which(HIPCC) is None and not os.path.exists(HIPCC), reason="hipcc not available")
def test_four_keys_stay_in_registers(tmp_path):
    exe = tmp_path / "keys_check"
    subprocess.check_call([HIPCC, "-O2", "-std=c++17", "--offload-arch=gfx950", "-x", "hip",
                           os.path.join(HERE, "native", "keys_check.hip"), "-o", str(exe)])
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    m = re.search(r"sequences (\d+) four (\d+) wrong (\d+)", out.stdout)
    assert m, out.stdout + out.stderr
    n, four, wrong = map(int, m.groups())
    assert n == 7 ** 8 and four > 100000
    assert out.returncode == 0 and wrong == 0, out.stdout
