"""Both sweeping kernels on strips below the heights that a caller can set, which only the autotuner's timing chooses
otherwise: every height it may choose, and one between them, against strips of 64 rows.

Fields and stage planes bit for bit; the sums of the centres are rounded by strip, at most N 2^-53 relative for N nodes
(1e-12 of the lattice is above that for every lattice here).  Sizes: a strip that ends at the lattice's edge, one with a
remainder of one row and of one column, plates, a batch of both; the reverse mode's record from such strips."""
import numpy as np
import pytest

from paper_1711_10984_amd import workloads as W

pytestmark = pytest.mark.gpu
HEIGHTS = [8, 10, 11, 12, 14]
FUSED, WAVE = 0, 2
LATTICES = {"whole": [(108, 112, 0)], "remainders": [(109, 113, 0)], "plates": [(131, 89, 1)],
            "batch": [(109, 113, 0), (131, 89, 1), (40, 20, 0)]}


def sim_of(shapes, prec, path):
    from paper_1711_10984_amd import lbm
    params, phi, c, f, drops = [], [], [], [], []
    for nx, ny, walls in shapes:
        g, p, q = W.random_state(nx, ny, nx)
        rng = np.random.default_rng(ny)
        params.append(dict(W.ACTIVE, nx=nx, ny=ny, walls=walls, tau=0.9, A0=1e-4))
        phi.append(p), c.append(q), f.append(g)
        drops.append([dict(x=rng.uniform(0, nx), y=rng.uniform(0, ny), R=12.0, Rs=5.0, ex=0.6, ey=0.8, active=1)
                      for _ in range(6)])
    return lbm, lbm.Sim(params, phi, c, drops, precision=prec, f_pre=f, path=path, graph_steps=4)


@pytest.mark.parametrize("prec", [0, 1, 2])
@pytest.mark.parametrize("path", [FUSED, WAVE])
@pytest.mark.parametrize("name", sorted(LATTICES))
def test_every_height_gives_the_same_fields(name, path, prec):
    shapes = LATTICES[name]
    lbm, want = sim_of(shapes, prec, path)
    want.set_seg_rows(64)
    stages = [want.stages(i) for i in range(want.n)]
    want.step(9)
    for h in HEIGHTS:
        _, sim = sim_of(shapes, prec, path)
        listed = sim.seg_rows
        lbm.lbm_debug_strips(sim.ctx, h)
        assert sim.running_rows == h and sim.seg_rows == listed
        assert sim.running_kernel == {FUSED: "k_step", WAVE: "k_wave"}[path]
        for i in range(sim.n):
            got = sim.stages(i)
            for k in got:
                assert np.array_equal(got[k], stages[i][k]), (h, i, k)
        sim.step(9)
        for i, (nx, ny, _) in enumerate(shapes):
            a, b = sim.fields(i), want.fields(i)
            for k in a:
                assert np.array_equal(a[k], b[k]), (h, i, k)
            for p, q in zip(sim.droplets(i), want.droplets(i)):
                assert abs(p["x"] - q["x"]) < 1e-12 * nx and abs(p["y"] - q["y"]) < 1e-12 * ny
        sim.close()
    want.close()


@pytest.mark.parametrize("path", [FUSED, WAVE])
def test_gradients_from_short_strips(path):
    """The derivatives take the droplets' centres from strip sums: they move by their rounding, as the fields' do not."""
    got = {}
    for h in (64, 8, 14):
        lbm, sim = sim_of([(109, 113, 0)], 0, path)
        lbm.lbm_debug_strips(sim.ctx, h)
        got[h] = (sim.adjoint_forward(0, 9, 4),) + sim.adjoint_backward()
        sim.close()
    J, dA0, dc0 = got[64]
    assert dA0 != 0.0
    for h in (8, 14):
        assert abs(got[h][0] - J) < 1e-12 * 109 and abs(got[h][1] - dA0) <= 1e-11 * abs(dA0)
        assert np.max(np.abs(got[h][2] - dc0)) <= 1e-11 * np.max(np.abs(dc0))


def test_heights_out_of_range():
    lbm, sim = sim_of([(109, 113, 0)], 0, WAVE)
    for rows in (7, 0, -1, 4097):
        with pytest.raises(lbm.LBMError):
            lbm.lbm_debug_strips(sim.ctx, rows)
    sim.close()
