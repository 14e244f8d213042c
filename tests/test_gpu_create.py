"""Instance preparation on the GPU against the oracle: candidate lists and the
nearest-neighbour tour's length, at the sizes and city sets where the selection
of the nearest cities changes its path."""
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


def _crowded(n, near, spread, seed=5):
    """`near` cities within `spread` of one point, the others far apart: one
    histogram bin of the selection then holds them all."""
    g = np.random.default_rng(seed)
    xy = g.random((n, 2)) * 60000.0 / np.sqrt(2.0)
    xy[:near] = 500.0 + g.random((near, 2)) * spread
    return xy


CASES = {
    "n3": (lambda: inputs.uniform(3), dict(cl=32)),
    "one_city_short_of_a_prefix": (lambda: inputs.uniform(161), dict(cl=32)),
    "prefix_of_every_other_city": (lambda: inputs.uniform(162), dict(cl=32)),
    "lists_of_64_and_a_prefix": (lambda: inputs.uniform(513), dict(cl=64)),
    "lattice_ties": (lambda: inputs.lattice(37), dict(cl=32)),
    "one_bin_refined": (lambda: _crowded(1300, 900, 40.0), dict(cl=32)),
    "hundreds_coincident": (lambda: inputs.coincident(1200, seed=3, dup=700), dict(cl=16)),
    "fewer_lds_neighbours": (lambda: inputs.uniform(5003), dict(cl=16)),
    "spm_short_list": (lambda: inputs.uniform(100), dict(cl=16, spm=True)),
    "spm_129_cities": (lambda: inputs.uniform(129), dict(cl=16, spm=True)),
    "spm_chunked_rows": (lambda: inputs.clustered(1111), dict(cl=32, spm=True, m=3)),
    "spm_coincident": (lambda: inputs.coincident(1200, seed=3, dup=700), dict(cl=16, spm=True)),
}


@pytest.mark.parametrize("name", list(CASES))
def test_candidates_and_nn_length(acs, name):
    make, kw = CASES[name]
    kw = dict(kw)
    xy = make()
    spm = kw.pop("spm", False)
    print(name, len(xy), flush=True)
    m = kw.pop("m", 8)
    col = acs.Colony(xy, m=m, memory=acs.ACS_SPM if spm else acs.ACS_DENSE, **kw)
    orc = oracle.Oracle(xy, m=m, memory=col.memory, **kw)
    assert np.array_equal(col.cand(), orc.cand())
    st, ref = col.stats(), orc.constants()
    assert st["nn_length"] == ref["lnn"]
    assert np.float32(st["tau0"]) == np.float32(ref["tau0"])
    for _ in range(2 if len(xy) < 2000 else 0):  # the fallback's lists, by the tours they give
        col.iterate(1)
        orc.iterate(1)
        assert np.array_equal(col.tours(), orc.tours())
    col.close()
    orc.close()


def test_refuses_distances_past_65535(acs):
    for xy in (np.array([[0.0, 0.0], [65600.0, 0.0], [1.0, 2.0]]),
               np.array([[0.0, 0.0], [60000.0, 60000.0], [1.0, 2.0]]),
               np.array([[0.0, 0.0], [1e200, 0.0], [1.0, 2.0]])):
        for memory in (acs.ACS_DENSE, acs.ACS_SPM):
            with pytest.raises(acs.AcsError) as e:
                acs.Colony(xy, cl=2, memory=memory)
            assert e.value.code == acs.ACS_E_UNSUPPORTED
