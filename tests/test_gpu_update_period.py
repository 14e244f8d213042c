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


# one ant, whose asynchronous construction is the sequential one; path 1: the
# ant's own updates, 2: through the updater wave; lanes 16: lane groups
@pytest.mark.parametrize("path,lanes,memory", [(1, 64, 0), (2, 64, 0), (1, 16, 0), (1, 64, 1),
                                               (2, 64, 1)])
@pytest.mark.parametrize("period", [0xFFFFFFFF, 0xFFFFFFF0, 0x80000001])
def test_asynchronous_periods_beyond_int32(acs, path, lanes, memory, period):
    xy = inputs.clustered(120)
    print(path, lanes, memory, period, flush=True)
    kw = dict(m=1, cl=12, memory=memory, seed=4)
    col = acs.Colony(xy, mode=acs.ACS_ASYNC_ATOMIC, update_path=path, lanes_per_ant=lanes,
                     local_update_period=period, **kw)
    orc = oracle.Oracle(xy, local_update_period=NEVER, **kw)
    for _ in range(4):
        col.iterate(1)
        orc.iterate(1)
        assert np.array_equal(col.tours(), orc.tours())
        assert np.array_equal(col.lengths(), orc.lengths())
        if memory:
            for x, y in zip(col.spm(), orc.spm()):
                assert np.array_equal(x, y)
        else:
            assert np.array_equal(col.tau(), orc.tau())
    col.close()
    orc.close()


@pytest.mark.parametrize("path", [1, 2])
def test_batch_periods_beyond_int32(acs, path):
    sizes = [120, 90]
    xys = [inputs.clustered(n) for n in sizes]
    b = acs.Batch(xys, m=1, cl=12, seed=4, local_update_period=0xFFFFFFFF, update_path=path,
                  lanes_per_ant=64)
    b.iterate(4)
    for i, xy in enumerate(xys):
        orc = oracle.Oracle(xy, m=1, cl=12, seed=4, instance=i, local_update_period=NEVER)
        orc.iterate(4)
        assert np.array_equal(b.lengths(i), orc.lengths())
        orc.close()
    b.close()
