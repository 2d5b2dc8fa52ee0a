"""The state read back in original order on both sides of the size at which
it goes through records (262,144 beads): set, sorted by an evaluation, and
read, every position (on the fixed-point lattice) and velocity comes back as
it was given, bit for bit, together and each alone."""
import numpy as np
import pytest
import torch

import gcme_workloads as W
from tests.gpu_common import make_engine

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [262143, 262144, 262147])
def test_state_comes_back(n):
    w = W.bulk("state", n, 7, 0.02, [0.4, 0.6], [[20.0, 25.0], [25.0, 30.0]], 1.5, 1.2, (16, 16, 16))
    eng = make_engine([w], "mixed")
    for sort in (False, True):
        if sort:
            eng.forces_energy()
        pos, vel, step = eng.get_state()
        eng.sync()
        assert step == 0
        assert np.array_equal(pos.t().cpu().numpy(), w.pos)
        assert np.array_equal(vel.t().cpu().numpy(), w.vel)
    only = torch.empty_like(pos)
    assert eng.lib.gcme_get_state(eng.h, only.data_ptr(), None, None) == 0
    eng.sync()
    assert torch.equal(only, pos)
    assert eng.lib.gcme_get_state(eng.h, None, only.data_ptr(), None) == 0
    eng.sync()
    assert torch.equal(only, vel)
    # the run goes on from the state: the sorted copy that held the records is made anew
    a = eng.forces_energy()["force"].clone()
    eng.sync()
    b = eng.forces_energy()["force"]
    eng.sync()
    assert torch.equal(a, b)
    eng.close()
