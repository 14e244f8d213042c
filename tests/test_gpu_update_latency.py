"""An ant that issues its own local updates goes on while they are in flight: a
step with updates is longer than one without by the instructions that issue
them, not by their round trip.  Two ants, so that nothing but one ant's chain of
steps sets the time.  Measured with one, two and four ants per wave: 1.40, 1.30
and 1.26 times the step without updates; 1.9 where the wave waits for the
result."""
import numpy as np
import pytest

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


@pytest.mark.parametrize("lanes", [64, 32, 16])
def test_step_does_not_wait_for_its_updates(acs, lanes):
    xy = inputs.uniform(500)

    def construct_ms(period):
        col = acs.Colony(xy, m=2, cl=16, mode=acs.ACS_ASYNC_ATOMIC, seed=5, lanes_per_ant=lanes,
                         update_path=1, local_update_period=period)
        col.iterate(5)
        ms = []
        for _ in range(15):
            col.iterate(1)
            ms.append(col.stats()["construct_ms"])
        col.close()
        return float(np.median(ms))

    every, never = construct_ms(1), construct_ms(1000)
    print(lanes, every, never, every / never, flush=True)
    assert every < 1.6 * never
