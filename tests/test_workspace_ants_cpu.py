"""acs_workspace_bytes with every number of ants the parameter's 32 bits hold: it
answers (numbers beyond what a launch takes are refused when a handle is
created, not here), with room for their tours at least.  The calls run in a
process of their own, which an arithmetic fault would end."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CODE = """
import ctypes, sys
sys.path.insert(0, %r)
from paper_1605_02669_amd import acs
lib = acs.load()
for m in list(range(1, 3000)) + [2**k + d for k in range(12, 31) for d in (-1, 0, 1, 15)] + [
        2**31 - 300, 2**31 - 256, 2**31 - 255, 2**31 - 1, 2**31, 2**31 + 1, 2**32 - 512,
        2**32 - 511, 2**32 - 300, 2**32 - 255, 2**32 - 1]:
    p = acs.make_params(cl=8, mode=%d, memory=%d)
    p.m = m
    out = ctypes.c_size_t()
    rc = lib.acs_workspace_bytes(100, ctypes.byref(p), ctypes.byref(out))
    assert rc == 0, (m, rc)
    assert m >= 2**31 or out.value > 4 * 100 * m, (m, out.value)
print("ok")
"""


@pytest.mark.parametrize("mode,memory", [(0, 0), (0, 1), (1, 0), (1, 1), (3, 0)])
def test_any_number_of_ants(mode, memory):
    r = subprocess.run([sys.executable, "-c", CODE % (ROOT, mode, memory)], capture_output=True,
                       text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.strip() == "ok", (r.returncode, r.stdout, r.stderr)
