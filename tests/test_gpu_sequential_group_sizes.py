"""Sequential construction with the group sizes that few cities or long update
periods choose (16 up to 128 in steps of 16), full groups, last groups of one ant
and of one short of full: equal to the oracle."""
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


# groups of 16 (n = 5, 79), 32 (80, 200), 48, 64 (period 2), 112 and 128 ants
@pytest.mark.parametrize("n,m,period", [(5, 33, 1), (79, 47, 1), (80, 65, 1), (200, 96, 1),
                                        (300, 95, 1), (200, 129, 2), (1000, 113, 1),
                                        (60, 200, 0xFFFFFFFF), (60, 200, 17), (40, 5000, 1)])
def test_group_sizes(acs, n, m, period):
    xy = inputs.uniform(n)
    print(n, m, period, flush=True)
    kw = dict(m=m, cl=min(16, n - 1), seed=11)
    col = acs.Colony(xy, mode=acs.ACS_SEQUENTIAL, local_update_period=period, **kw)
    orc = oracle.Oracle(xy, mode=oracle.SEQUENTIAL, local_update_period=min(period, 0x7FFFFFFF),
                        **kw)
    for _ in range(2):
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
