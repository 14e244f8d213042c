"""acs_candidates writes into the caller's buffer and takes no host memory of its own
that grows with the instance: it answers in a process that can map no more
(where an allocation of 20 MB would end the process by an exception), with the
lists of an ordinary call, whole and in every part of them."""
import os
import subprocess
import sys

import numpy as np
import pytest

import oracle
from paper_1605_02669_amd import inputs

pytestmark = pytest.mark.gpu
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CODE = """
import resource, sys
sys.path.insert(0, %r)
import numpy as np
from paper_1605_02669_amd import acs, inputs
n, cl = 20000, 64
col = acs.Colony(inputs.uniform(n), m=8, cl=cl, mode=acs.ACS_ASYNC_ATOMIC, torch_memory=False)
want, got = col.cand(), np.zeros((n, cl), np.int32)
used = 1024 * int([l for l in open("/proc/self/status") if l.startswith("VmSize")][0].split()[1])
hard = resource.getrlimit(resource.RLIMIT_AS)[1]
resource.setrlimit(resource.RLIMIT_AS, (used + (8 << 20), hard))
rc = acs.load().acs_candidates(col.h, acs._ptr(got), got.size)
resource.setrlimit(resource.RLIMIT_AS, (hard, hard))
assert rc == 0 and np.array_equal(got, want), rc
col.close()
print("ok")
"""


@pytest.fixture(scope="module")
def acs():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1605_02669_amd import acs as mod
    mod.load()
    return mod


def test_no_host_memory(acs):
    r = subprocess.run([sys.executable, "-c", CODE % ROOT], capture_output=True, text=True,
                       timeout=100)
    assert r.returncode == 0 and r.stdout.strip() == "ok", (r.returncode, r.stdout, r.stderr)


# 4096 records are the last part: around it, one and several parts before it
@pytest.mark.parametrize("n,cl", [(3, 2), (64, 63), (64, 64), (65, 64), (171, 24), (1400, 4),
                                  (1000, 33)])
def test_lists(acs, n, cl):
    xy = inputs.uniform(n)
    col, orc = acs.Colony(xy, m=2, cl=cl, mode=acs.ACS_ASYNC_ATOMIC), oracle.Oracle(xy, m=2, cl=cl)
    assert np.array_equal(col.cand(), orc.cand())
    col.close()
    orc.close()


# wherever the lists' place holds something else after creation (updates' counts,
# the grid barrier's words): the lists between iterations, and iterations as if
# they had not been read
@pytest.mark.parametrize("mode,memory,m,period", [
    (0, 0, 200, 1), (0, 0, 200, 3), (0, 0, 1100, 1), (0, 0, 1100, 4), (0, 1, 40, 1), (1, 0, 1, 1),
    (1, 0, 1, 5), (2, 0, 1, 1), (1, 1, 1, 1), (3, 0, 20, 1)])
def test_lists_between_iterations(acs, mode, memory, m, period):
    xy = inputs.uniform(300)
    kw = dict(m=m, cl=24, mode=mode, memory=memory, seed=4, local_update_period=period)
    read, left = acs.Colony(xy, **kw), acs.Colony(xy, **kw)
    orc = oracle.Oracle(xy, m=1, cl=24)
    for _ in range(3):
        assert np.array_equal(read.cand(), orc.cand())
        read.iterate(1)
        left.iterate(1)
        assert np.array_equal(read.tours(), left.tours())
        if memory == 0:
            assert np.array_equal(read.tau(), left.tau())
    assert np.array_equal(read.cand(), orc.cand())
    for c in (read, left, orc):
        c.close()
