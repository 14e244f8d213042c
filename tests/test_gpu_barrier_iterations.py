"""The synchronous kernels' grid barrier over more iterations than its words go
between two clearings (2^14): a long run equals the oracle's."""
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


# twenty blocks over all XCDs; dense: n * cl too small for the pheromone in LDS
@pytest.mark.parametrize("memory", [0, 1])
def test_barrier_across_its_clearings(acs, memory):
    xy = inputs.uniform(5)
    kw = dict(m=20, cl=2, memory=memory, seed=9)
    col, orc = acs.Colony(xy, **kw), oracle.Oracle(xy, **kw)
    for k in (16380, 8, 600):
        print(memory, k, flush=True)
        col.iterate(k)
        orc.iterate(k)
        assert np.array_equal(col.tours(), orc.tours())
        assert np.array_equal(col.lengths(), orc.lengths())
        if memory:
            for x, y in zip(col.spm(), orc.spm()):
                assert np.array_equal(x, y)
        else:
            assert np.array_equal(col.tau(), orc.tau())
    col.close()
    orc.close()
