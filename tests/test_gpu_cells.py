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
# 131,072, where the one-launch scan ends; more beads than the one-block sort
# takes.  FP64, TOL as above.
GRIDS = {4095: (15, 13, 21), 4096: (16, 16, 16), 4100: (10, 10, 41), 8192: (16, 16, 32),
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
