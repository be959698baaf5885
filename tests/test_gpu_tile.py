"""The tiled kernel that the fused path takes for small lattices: against the oracle and the strip kernels.

FP64 evaluates the oracle's expressions in the oracle's order, and in every precision the kernels of all paths share
their arithmetic, so fields are compared bit for bit.  The centres' sums are carried in twice the working precision
and rounded once, so they do not depend on how the steps are grouped into calls and graphs (also bit for bit); the
strip kernels' plain sums differ from them by rounding, at most N 2^-53 relative for N nodes (1e-12 of the lattice
is above that for every lattice here)."""
import numpy as np
import pytest

from oracle import Drop, OracleSim, Params
from paper_1711_10984_amd import workloads as W

pytestmark = pytest.mark.gpu
FIELDS = ("f", "phi", "c", "n", "ux", "uy")


def _lbm():
    from paper_1711_10984_amd import lbm
    return lbm


def random_case(nx, ny, ndrop, walls=0, advection=0, seed=3):
    """Random fields with droplets all over the lattice, so that many tiles hold nodes of each."""
    f, phi, c = W.random_state(nx, ny, seed)
    rng = np.random.default_rng(seed + 1)
    drops = [dict(x=rng.uniform(0, nx), y=rng.uniform(0, ny), R=min(nx, ny) / 3.0, Rs=min(nx, ny) / 7.0, ex=0.6, ey=0.8,
                  active=int(k != 1)) for k in range(ndrop)]
    p = dict(W.ACTIVE, nx=nx, ny=ny, A0=1e-4, gamma=0.01, c0=0.02, Gamma=0.05, tau=0.8, walls=walls, advection=advection)
    return p, phi, c, drops, f


def sim_of(case, precision=0, path=0, graph_steps=0, step=2):
    p, phi, c, drops, f = case
    return _lbm().Sim([p], [phi], [c], [drops], precision=precision, f_pre=[f], step=step, path=path,
                      graph_steps=graph_steps)


def same_fields(a, b, what):
    for k in FIELDS:
        assert np.array_equal(a[k], b[k]), (what, k, float(np.max(np.abs(a[k] - b[k]))))


def near_centres(a, b, L):
    for p, q in zip(a, b):
        assert abs(p["x"] - q["x"]) < 1e-12 * L and abs(p["y"] - q["y"]) < 1e-12 * L


# the smallest lattice of each tile shape and one node less (which strips take); tiles that end at the lattice's
# edge, or one node before or after it; the last sizes of the first two shapes (256 tiles) and beyond
SIZES = [(21, 13), (20, 13), (21, 12), (48, 32), (49, 33), (47, 31), (256, 128), (257, 128), (256, 256), (257, 256)]


@pytest.mark.parametrize("walls,advection", [(0, 0), (1, 0), (0, 1), (1, 1)])
@pytest.mark.parametrize("shape", SIZES)
def test_fields_are_the_oracles_bit_for_bit(shape, walls, advection):
    nx, ny = shape
    case = random_case(nx, ny, 3, walls, advection)
    p, phi, c, drops, f = case
    sim = sim_of(case)
    ref = OracleSim(Params(**p), phi, c, [Drop(**d) for d in drops], f_pre=f, step=2)
    got, want = sim.stages(), ref.stages()
    for k in want:
        assert np.array_equal(got[k], want[k]), (shape, k)
    sim.step(6)
    ref.run(6)
    same_fields(sim.fields(), ref.fields(), shape)
    for g, r in zip(sim.droplets(), ref.drops()):
        assert abs(g["x"] - r.x) < 1e-12 * nx and abs(g["y"] - r.y) < 1e-12 * nx
    sim.close()


@pytest.mark.parametrize("precision", [0, 1, 2])
@pytest.mark.parametrize("ndrop", [0, 1, 9, 16, 17])
def test_droplet_counts_and_precisions_match_the_strips(ndrop, precision):
    """0 and 1 droplets, more than the workgroup's eight wavefronts, the most tiles take, and one more."""
    case = random_case(97, 61, ndrop, seed=11 + ndrop)
    a, b = sim_of(case, precision), sim_of(case, precision, path=2)
    for s in (a, b):
        s.step(9)
    same_fields(a.fields(), b.fields(), (ndrop, precision))
    near_centres(a.droplets(), b.droplets(), 97)
    a.close()
    b.close()


@pytest.mark.parametrize("shape", [(64, 64), (500, 500)])
def test_grouping_of_the_steps_changes_nothing(shape):
    """One call, calls of single steps, a replayed graph and a remainder: fields and centres bit for bit.  500 x 500
    has 512 of the largest tiles, more than one chunk of presence bits, and droplets over more than 64 of them."""
    nx, ny = shape
    case = random_case(nx, ny, 2, seed=5)
    one = sim_of(case)
    one.step(27)
    want, centres = one.fields(), one.droplets()
    singles = sim_of(case)
    for _ in range(27):
        singles.step(1)
    graphs = sim_of(case, graph_steps=10)
    graphs.step(3)
    graphs.step(24)
    for s in (singles, graphs):
        same_fields(s.fields(), want, shape)
        assert s.droplets() == centres and s.step_count == 29
        s.close()
    strips = sim_of(case)
    strips.set_seg_rows(64)  # the caller asks for strips
    strips.step(27)
    same_fields(strips.fields(), want, shape)
    near_centres(strips.droplets(), centres, nx)
    strips.close()
    one.close()


def test_batch_of_uneven_lattices_matches_single_runs():
    cases = [random_case(64, 48, 2, seed=21), random_case(31, 90, 0, walls=1, seed=22), random_case(90, 31, 1, seed=23)]
    lbm = _lbm()
    batch = lbm.Sim([c[0] for c in cases], [c[1] for c in cases], [c[2] for c in cases], [c[3] for c in cases],
                    f_pre=[c[4] for c in cases], step=2, graph_steps=4)
    batch.step(11)
    for i, case in enumerate(cases):
        alone = sim_of(case)
        alone.step(11)
        same_fields(batch.fields(i), alone.fields(), i)
        assert batch.droplets(i) == alone.droplets()
        alone.close()
    batch.close()
