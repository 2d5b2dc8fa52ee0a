"""Cell order and cluster enumeration against the FP64 oracle: every cell
shape of the tuning (flat cells, odd columns counted downwards), axes of one
and two cells, odd and even column heights, clusters that cross from one
column to the next (ragged bead counts), and a box with an empty gap along z,
where such a cluster would span the gap."""
import numpy as np
import pytest

import gcme_workloads as W
from tests.gpu_common import make_engine, oracle_eval, rel_rms

pytestmark = pytest.mark.gpu

# force relative RMS: FP64 sums of about 1e3 pairs at 1e-16; single precision
# 2^-24 per pair term, the bound the other parity tests use
TOL = {"fp64": 1e-9, "mixed": 1e-5}


def gap_box(n, box, fill, seed):
    """n beads in the lower `fill` of the box's height."""
    w = W.small_bulk(N=n, seed=seed, box=box, rc=2.0, grid=(16, 16, 32))
    pos = w.pos.copy()
    pos[:, 2] *= fill
    w.pos = W.lattice_positions(pos / np.asarray(box), box)
    return w


CASES = {
    "cube": lambda: W.small_bulk(N=403, seed=3, box=(5.4, 5.5, 5.6), rc=2.0, grid=(16, 16, 16)),
    "one_cell_axes": lambda: W.small_bulk(N=251, seed=4, box=(4.0, 4.1, 12.3), rc=2.0, grid=(16, 16, 32)),
    "flat": lambda: W.small_bulk(N=517, seed=5, box=(12.1, 11.3, 4.2), rc=2.0, grid=(32, 32, 16)),
    "gap": lambda: gap_box(509, (6.3, 7.1, 21.0), 0.3, 6),
}


@pytest.mark.parametrize("direct", [0, 3])
@pytest.mark.parametrize("n", [1, 2, 3, 4])
@pytest.mark.parametrize("case", sorted(CASES))
def test_cells_against_oracle(case, n, direct):
    w = CASES[case]()
    ref = oracle_eval(w)
    for prec in ("fp64", "mixed"):
        for ci in (2, 4, 8):
            eng = make_engine([w], prec, tuning=dict(cells_per_cutoff=n, beads_per_cluster=ci, charges_per_cluster=ci,
                                                     direct_pairs=direct, list_slack_pct=400))
            for ev in (True, False):
                out = eng.forces_energy(energy=ev, virial=ev)
                eng.sync()
                err = rel_rms(out["force"].t().cpu().numpy(), ref["F"])
                assert err < TOL[prec], (case, n, prec, ci, ev, err)
            eng.close()


# cells of the grid (rc = 1, one cell per cutoff across, two along z): the
# scan's blocks of 4,096 cells and the cells beside them, and both sides of
# 24,576, where the bucket sort ends, and of 131,072, where the one-launch scan
# does; more beads than the one-block sort
# takes.  FP64, TOL as above.
GRIDS = {4095: (15, 13, 21), 4096: (16, 16, 16), 4100: (10, 10, 41), 8192: (16, 16, 32), 24576: (32, 32, 24),
         25600: (32, 32, 25),
         131040: (63, 65, 32), 131072: (64, 64, 32), 133120: (65, 64, 32)}


@pytest.mark.parametrize("cells", sorted(GRIDS))
def test_scan_sizes_against_oracle(cells):
    nx, ny, nz = GRIDS[cells]
    assert nx * ny * nz == cells
    w = W.small_bulk(N=4203, seed=7, box=(nx + 0.2, ny + 0.2, (nz + 0.4) / 2), rc=1.0, grid=(64, 64, 32))
    ref = oracle_eval(w)
    eng = make_engine([w], "fp64", tuning=dict(cells_per_cutoff=1, direct_pairs=3))
    for _ in range(2):  # again from the counts that the first sort left cleared
        out = eng.forces_energy(energy=False, virial=False)
        eng.sync()
        err = rel_rms(out["force"].t().cpu().numpy(), ref["F"])
        assert err < TOL["fp64"], (cells, err)
    eng.close()


# Cluster sizes by the number of beads (charged fraction f): up to 6,144 beads
# clusters of 2, up to 16,384 of 4, above of 8; up to 8,192 charges of 2, above
# of 4.  Bit-identical to the same sizes given, and the general sizes agree to
# FP64 sums (TOL).
SIZES = [(6144, 0.2, 2, 2), (6145, 0.2, 4, 2), (16384, 0.5, 4, 2), (16384, 0.51, 4, 4), (16385, 0.2, 8, 2)]


@pytest.mark.parametrize("n,frac,cg,cq", SIZES)
def test_default_cluster_sizes(n, frac, cg, cq):
    box = (n / 2.5) ** (1.0 / 3.0)
    w = W.small_bulk(N=n, seed=8, charged_frac=frac, box=(box, 1.01 * box, 0.99 * box), rc=2.0, grid=(36, 36, 36))
    F = []
    for tuning in (None, dict(beads_per_cluster=cg, charges_per_cluster=cq),
                   dict(beads_per_cluster=8, charges_per_cluster=4)):
        eng = make_engine([w], "fp64", tuning=tuning)
        out = eng.forces_energy(energy=True, virial=True)
        eng.sync()
        F.append(out["force"].cpu().numpy())
        eng.close()
    np.testing.assert_array_equal(F[0], F[1])
    assert rel_rms(F[0], F[2]) < TOL["fp64"]


def test_given_cluster_sizes_stand():
    """A size once given is kept, also where it is the one that was reported."""
    w = W.small_bulk(N=700, seed=9, box=(6.6, 6.5, 6.7), rc=2.4, grid=(24, 24, 24))
    eng = make_engine([w], "mixed")
    auto = eng.forces_energy()["force"].clone()
    t = eng.tuning()
    eng.set_tuning(beads_per_cluster=t["beads_per_cluster"], charges_per_cluster=t["charges_per_cluster"])
    given = eng.forces_energy()["force"].clone()
    eng.sync()
    eng.close()
    fresh = make_engine([w], "mixed", tuning=dict(beads_per_cluster=8, charges_per_cluster=4))
    ref = fresh.forces_energy()["force"]
    fresh.sync()
    assert t["beads_per_cluster"] == 8 and t["charges_per_cluster"] == 4
    np.testing.assert_array_equal(given.cpu().numpy(), ref.cpu().numpy())
    assert rel_rms(auto.cpu().numpy(), ref.cpu().numpy()) < TOL["mixed"]
    fresh.close()


@pytest.mark.parametrize("direct", [0, 3])
@pytest.mark.parametrize("axis", [0, 1, 2])
@pytest.mark.parametrize("precision", ["mixed", "fp64"])
def test_cluster_across_the_whole_axis(axis, direct, precision):
    """One cluster with beads half the axis away on either side, 2^31 and
    2^31 - 1 units of the fixed-point lattice from its first: its bounding box
    is the axis to the last unit."""
    w = W.small_bulk(N=8, seed=10, box=(10.0, 10.0, 10.0), rc=2.0, charged_frac=0.5, grid=(24, 24, 24))
    f = np.full((8, 3), 0.04)
    f[:, (axis + 1) % 3] += np.linspace(0.0, 0.05, 8)
    f[:, (axis + 2) % 3] += np.linspace(0.05, 0.0, 8)
    f[:, axis] = np.array([0.0, 2.0**31, 2.0**31 - 1, 1e8, 2e8, 3e8, 2.0**31 - 2e8, 2.0**31 - 3e8]) / 2.0**32
    f[0, (axis + 1) % 3] = f[0, (axis + 2) % 3] = 0.0  # (the first in cell order)
    w.pos = W.lattice_positions(f, w.box)
    ref = oracle_eval(w)
    eng = make_engine([w], precision, tuning=dict(beads_per_cluster=8, charges_per_cluster=8, direct_pairs=direct,
                                                  list_slack_pct=1000))
    out = eng.forces_energy()
    eng.sync()
    assert rel_rms(out["force"].t().cpu().numpy(), ref["F"]) < TOL[precision]
    eng.close()


# The stream layout that is taken while none is given (three branches from 1,000
# beads within a bead's cutoff on, or with column clusters for the charges)
# changes no result: forces are integer sums.
@pytest.mark.parametrize("n,box,tuning", [(4000, 6.3, {}), (4000, 6.5, {}), (3000, 10.6, dict(half_pairs=10)),
                                          (3000, 10.6, dict(half_pairs=2))])
def test_layouts_agree(n, box, tuning):
    w = W.small_bulk(N=n, seed=11, box=(box, box, box), rc=2.5, grid=(24, 24, 24))
    states = []
    for layout in (None, 0, 2, None):
        eng = make_engine([w], "mixed", tuning=dict(tuning) if layout is None else dict(tuning, stream_layout=layout))
        eng.step(10)
        if layout is None and states:  # given between two runs
            eng.set_tuning(stream_layout=2)
            eng.set_state(w.pos, w.type, w.z, w.vel)
            eng.step(10)
        pos, vel, _ = eng.get_state()
        eng.sync()
        states.append((pos.cpu().numpy(), vel.cpu().numpy()))
        eng.close()
    for s in states[1:]:
        np.testing.assert_array_equal(s[0], states[0][0])
        np.testing.assert_array_equal(s[1], states[0][1])
