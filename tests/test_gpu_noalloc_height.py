"""lbm_step_noalloc and lbm_step on strips of the height that lbm_noalloc_rows tells: the same bits, centres included.

The sizes: the fixed height, the lowest that strips of a context can have (8 rows), heights below and above 16, remainders
of a strip in x and y, plates, in each storage type; 40 rows because shorter strips' sums of 60 droplets do not fit."""
import numpy as np
import pytest

from paper_1711_10984_amd import workloads as W
from test_gpu_noalloc_rows import noalloc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,walls,prec,ndrop", [(255, 256, 0, 0, 5), (251, 200, 1, 2, 5), (600, 600, 0, 0, 5),
                                                    (700, 701, 1, 0, 5), (900, 901, 0, 0, 5), (900, 901, 1, 1, 5),
                                                    (900, 901, 0, 2, 5), (1300, 1301, 0, 0, 5), (1300, 1301, 0, 1, 5),
                                                    (1300, 1301, 1, 2, 5), (70200, 208, 0, 1, 5), (70200, 208, 0, 1, 60)])
def test_the_same_bits_at_the_same_height(nx, ny, walls, prec, ndrop):
    from paper_1711_10984_amd import lbm
    rng = np.random.default_rng(nx + ny + prec)
    p = dict(W.ACTIVE, nx=nx, ny=ny, walls=walls, tau=0.9)
    phi = 0.3 * rng.standard_normal((ny, nx)) - 0.3
    c = 0.05 + 0.01 * rng.standard_normal((ny, nx))
    drops = [dict(x=rng.uniform(0, nx), y=rng.uniform(0, ny), R=ny / 4.0, Rs=ny / 9.0, ex=0.6, ey=-0.8, active=1)
             for _ in range(ndrop)]
    sim = lbm.Sim([p], [phi], [c], [drops], precision=prec, path=lbm.LBM_PATH_WAVE, graph_steps=0)
    rows = lbm.lbm_noalloc_rows(lbm.make_config(p, prec), len(drops))
    lbm.lbm_debug_strips(sim.ctx, rows)
    nsteps = 6
    got_phi, got_c, at = noalloc(lbm, p, phi, c, sim.droplets(), prec, nsteps)
    sim.step(nsteps)
    want = sim.fields()
    assert np.array_equal(got_phi, want["phi"]) and np.array_equal(got_c, want["c"])
    assert at == [(d["x"], d["y"]) for d in sim.droplets()]
    sim.close()
