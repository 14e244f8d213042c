"""Update periods up to the largest an unsigned 32-bit word holds: a period of
at least n means that only the closing edges are updated, whatever its value."""
import numpy as np
import pytest

import oracle
from paper_1605_02669_amd import inputs

pytestmark = pytest.mark.gpu

NEVER = 0x7FFFFFFF  # the oracle's largest


@pytest.fixture(scope="module")
def acs():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1605_02669_amd import acs as mod
    mod.load()
    return mod


# 70 ants: pheromone in LDS (n * cl * 4 bytes hold the blocks' words); cl = 2
# and m = 1025: the records' pheromone
@pytest.mark.parametrize("n,m,cl", [(120, 70, 12), (121, 70, 12), (120, 70, 2), (60, 1025, 6)])
@pytest.mark.parametrize("period", [0xFFFFFFFF, 0xFFFFFFF0, 0x80000001])
def test_synchronous_periods_beyond_int32(acs, n, m, cl, period):
    xy = inputs.clustered(n)
    print(n, m, cl, period, flush=True)
    kw = dict(m=m, cl=cl, seed=3)
    col = acs.Colony(xy, local_update_period=period, **kw)
    orc = oracle.Oracle(xy, local_update_period=NEVER, **kw)
    for _ in range(4):
        col.iterate(1)
        orc.iterate(1)
        assert np.array_equal(col.tours(), orc.tours())
        assert np.array_equal(col.lengths(), orc.lengths())
        assert np.array_equal(col.tau(), orc.tau())
    col.close()
    orc.close()
