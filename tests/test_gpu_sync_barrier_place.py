"""Dense synchronous handles whose grid barrier's words take the place of the lists or of the
eta^beta table once the handle is built: tours, lengths, pheromone and candidate
lists equal the oracle's, also where the table was full up to the largest
distance (the last city 65535 away), over calls and with another handle between
them."""
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


@pytest.mark.parametrize("far", [False, True])
@pytest.mark.parametrize("n,m,cl,period", [(3, 1, 2, 1), (20, 40, 2, 1), (61, 256, 12, 1),
                                           (61, 300, 4, 3), (198, 150, 1, 1), (300, 1100, 32, 1),
                                           (400, 1025, 8, 2)])
def test_words_in_the_tables_place(acs, n, m, cl, period, far):
    print(n, m, cl, period, far, flush=True)
    xy = inputs.uniform(n)
    if far:
        # (nobody else farther from the last city than the first is: 65535 is the limit)
        xy = 1000 + np.floor(xy / xy.max() * 9000) * (1, 0.1)
        xy[0], xy[n - 1] = (0, 0), (65535, 0)
    kw = dict(m=m, cl=cl, seed=9, local_update_period=period)
    col, other, orc = acs.Colony(xy, **kw), acs.Colony(inputs.uniform(50)), oracle.Oracle(xy, **kw)
    for k in (1, 2):
        col.iterate(k)
        other.iterate(1)
        orc.iterate(k)
        assert np.array_equal(col.tours(), orc.tours())
        assert np.array_equal(col.lengths(), orc.lengths())
        assert np.array_equal(col.tau(), orc.tau())
        assert np.array_equal(col.cand(), orc.cand())
    for c in (col, other, orc):
        c.close()
