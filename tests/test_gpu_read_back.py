"""lbm_fields: what it returns at step 0 is the initial state as stored, to the bit, however the read-back is cut.

Read-backs above 512 KB go in chunks of that: the sizes are the smallest lattice, one chunk full (4681 nodes of 14
planes), two nodes beyond it, many chunks with a remainder, and single planes beyond a chunk."""
import numpy as np
import pytest

from paper_1711_10984_amd import workloads as W

pytestmark = pytest.mark.gpu
WT = np.array([4 / 9] + [1 / 9] * 4 + [1 / 36] * 4)[:, None, None]


def as_stored(f, prec):
    if prec == 0:
        return f
    w = np.float32(WT)
    if prec == 1:
        return (f - w.astype(np.float64)).astype(np.float32).astype(np.float64) + w.astype(np.float64)
    return ((f.astype(np.float32) - w).astype(np.float16).astype(np.float32) + w).astype(np.float64)


def make(nx, ny, prec, walls, batch=False):
    from paper_1711_10984_amd import lbm
    f, phi, c = W.random_state(nx, ny, 5)
    p = dict(W.ACTIVE, nx=nx, ny=ny, walls=walls)
    if batch:  # the lattice behind another one
        g, phi2, c2 = W.random_state(40, 30, 6)
        q = dict(W.ACTIVE, nx=40, ny=30)
        sim = lbm.Sim([q, p], [phi2, phi], [c2, c], [[], []], precision=prec, f_pre=[g, f])
    else:
        sim = lbm.Sim([p], [phi], [c], [[]], precision=prec, f_pre=[f])
    return lbm, sim, f, phi, c


@pytest.mark.parametrize("prec", [0, 1, 2])
@pytest.mark.parametrize("nx,ny,walls", [(3, 3, 0), (3, 3, 1), (31, 151, 0), (3, 1561, 1), (1561, 3, 0), (257, 250, 1)])
def test_initial_state_comes_back(nx, ny, walls, prec):
    lbm, sim, f, phi, c = make(nx, ny, prec, walls, batch=nx == 257)
    i = sim.n - 1
    held = lambda a: a if prec == 0 else a.astype(np.float32).astype(np.float64)
    got = sim.fields(i)
    assert np.array_equal(got["f"], as_stored(f, prec))
    assert np.array_equal(got["phi"], held(phi)) and np.array_equal(got["c"], held(c))
    # single planes, and the same values from them
    for k in ("f", "phi", "n", "uy"):
        out = np.full_like(got[k], np.nan)
        lbm.lbm_fields(sim.ctx, i, **{"f_pre" if k == "f" else k: out})
        assert np.array_equal(out, got[k]), k
    # n = sum f in the precision of the arithmetic: nine terms, 9 ulp of n (FP16 storage sums its rounded values)
    eps = 2.0 ** -52 if prec == 0 else 2.0 ** -23
    assert np.max(np.abs(got["n"] - got["f"].sum(0)) / got["n"]) < 9 * eps
    sim.close()


def test_one_plane_in_several_chunks_and_its_last_value_not_finite():
    from paper_1711_10984_amd import lbm
    nx, ny = 601, 500  # 300 500 nodes, 65 536 to a chunk
    f, phi, c = W.random_state(nx, ny, 7)
    phi[-1, -1] = np.inf
    sim = lbm.Sim([dict(W.ACTIVE, nx=nx, ny=ny)], [phi], [c], [[]], f_pre=[f])
    out = np.empty((ny, nx))
    assert lbm.lbm_fields(sim.ctx, 0, c=out) == lbm.LBM_OK
    assert np.array_equal(out, c)
    assert lbm.lbm_fields(sim.ctx, 0, phi=out) == lbm.LBM_E_UNSTABLE
    assert np.array_equal(out, phi)
    sim.close()
