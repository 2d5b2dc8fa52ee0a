"""New pair strengths and radii on a live context (only its type-pair tables
and constants are sent again; mesh, cells and captured step graphs stay)
against a context made with them, bit for bit: evaluation, parameter
derivatives and a run of steps, one replica and several, for each thing that
may change alone; and changes that need the whole plan."""
import dataclasses

import numpy as np
import pytest

import gcme_workloads as W
from paper_2403_08148_amd import GCMe, params_from_workload

pytestmark = pytest.mark.gpu

WS = [W.small_bulk(N=n, seed=20 + n, box=b, rc=2.0, grid=(16, 16, 16))
      for n, b in ((300, (4.9, 5.0, 5.1)), (211, (4.4, 4.3, 4.5)))]
NEW = {
    "A": lambda p: dict(A=1.1 * np.asarray(p.A)),
    "a": lambda p: dict(a=np.asarray(p.a) * 1.05),
    "sigma": lambda p: dict(sigma=np.asarray(p.sigma) * 0.95),
    "all": lambda p: dict(A=0.9 * np.asarray(p.A), a=np.asarray(p.a) * 0.97, sigma=np.asarray(p.sigma) * 1.02),
    "nothing": lambda p: {},
    "lB": lambda p: dict(lB=1.3, A=1.2 * np.asarray(p.A)),  # the whole plan
    "dt": lambda p: dict(dt=0.01),
    "beta": lambda p: dict(beta=1.0),
}


def state_of(eng):
    ws = WS[:eng.R]
    eng.set_state(*[np.concatenate([getattr(w, f) for w in ws]) for f in ("pos", "type", "z", "vel")])


def results(eng):
    out = eng.forces_energy(adjoint=True)
    eng.step(3)
    pos, vel, _ = eng.get_state()
    eng.sync()
    return [t.cpu().numpy() for t in list(out.values()) + [pos, vel]]


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("replicas", [1, 2])
@pytest.mark.parametrize("what", sorted(NEW))
def test_new_parameters_on_a_live_context(what, replicas, precision):
    old = [params_from_workload(w) for w in WS[:replicas]]
    new = [dataclasses.replace(p, **NEW[what](p)) for p in old]
    n = [w.N for w in WS[:replicas]]
    live = GCMe(n, precision=precision, seed=4)
    for r, p in enumerate(old):
        live.set_params(p, r)
    state_of(live)
    live.step(12)  # captures and replays every step graph
    live.sync()
    state_of(live)
    live.step(1)
    live.sync()
    for r, p in enumerate(new):
        live.set_params(p, r)
    # (the state's order within cells is kept from the run, so both start from the state anew)
    fresh = GCMe(n, precision=precision, seed=4)
    for r, p in enumerate(new):
        fresh.set_params(p, r)
    state_of(fresh)
    if what in ("A", "a", "sigma", "all", "nothing"):
        # without set_state the plan is not built again: an evaluation at the same positions,
        # summed in another order, then the same from the same state
        pos = np.concatenate([w.pos for w in WS[:replicas]])
        got = live.forces_energy(pos=pos)["force"].cpu().numpy()
        ref = fresh.forces_energy(pos=pos)["force"].cpu().numpy()
        tol = 1e-12 if precision == "fp64" else 1e-5
        assert np.linalg.norm(got - ref) < tol * np.linalg.norm(ref)
        state_of(fresh)
    state_of(live)
    for r, p in enumerate(old):
        live.set_params(p, r)
    for r, p in enumerate(new):
        live.set_params(p, r)  # back and forth: the last ones count
    for x, y in zip(results(live), results(fresh)):
        assert np.array_equal(x, y)
    live.close()
    fresh.close()
