"""The sequential schedule at the edges of its groups of 128 ants, with many
conflicts inside a group, with rows that share a slot of the conflict table
(n > 4096), with more ants than current cities kept in LDS, and with visited
bitmaps in global memory."""
import numpy as np
import pytest

import oracle
from paper_1605_02669_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def acs():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1605_02669_amd import acs as mod
    mod.load()
    return mod


@pytest.mark.parametrize("n,m,cl,period", [(5, 128, 4, 1), (23, 129, 8, 1), (300, 257, 40, 1),
                                           (90, 300, 12, 4), (4500, 3, 8, 1), (12, 4097, 6, 1),
                                           (1300, 800, 16, 1)])
def test_sequential_groups(acs, n, m, cl, period):
    xy = inputs.uniform(n)
    print(n, m, cl, period, flush=True)
    iters = 1 if n * m > 10 ** 6 else 2
    col = acs.Colony(xy, m=m, cl=cl, seed=8, mode=acs.ACS_SEQUENTIAL, local_update_period=period)
    orc = oracle.Oracle(xy, m=m, cl=cl, seed=8, mode=oracle.SEQUENTIAL,
                        local_update_period=period)
    for _ in range(iters):
        col.iterate(1)
        orc.iterate(1)
        assert np.array_equal(col.tours(), orc.tours())
        assert np.array_equal(col.lengths(), orc.lengths())
        assert np.array_equal(col.tau(), orc.tau())
    st, oc = col.stats(), orc.counts()
    for k in ("steps", "greedy", "roulette", "fallback"):
        assert st[k] == oc[k], k
    col.close()
    orc.close()
