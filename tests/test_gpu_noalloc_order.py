"""lbm_step_noalloc lists each strip once, whatever the droplets: the same bits as lbm_step on strips of the same height.

The sizes: one strip, fewer strips than runs, one lane a droplet and several (1, 5, 64, 256 droplets), a last run that is
short or empty, runs of 512 strips (the longest that are ordered by distance), of 511.25 and of 512.5 (not ordered)."""
import numpy as np
import pytest

from paper_1711_10984_amd import workloads as W
from test_gpu_noalloc_rows import noalloc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,walls,prec,ndrop", [(54, 40, 0, 0, 64), (100, 90, 1, 0, 256), (251, 200, 0, 1, 1),
                                                    (600, 600, 1, 0, 256), (1300, 1301, 0, 2, 64),
                                                    (1300, 1301, 0, 1, 256), (2048, 2048, 0, 1, 256),
                                                    (220860, 16, 0, 1, 5), (221184, 16, 0, 1, 64), (221400, 16, 0, 1, 64)])
def test_the_same_bits_in_any_order(nx, ny, walls, prec, ndrop):
    from paper_1711_10984_amd import lbm
    rng = np.random.default_rng(nx + ndrop)
    p = dict(W.ACTIVE, nx=nx, ny=ny, walls=walls, tau=0.9)
    phi = 0.3 * rng.standard_normal((ny, nx)) - 0.3
    c = 0.05 + 0.01 * rng.standard_normal((ny, nx))
    R = min(ny / 4.0, 12.0)
    drops = [dict(x=rng.uniform(0, nx), y=rng.uniform(R, ny - R), R=R, Rs=R / 2, ex=0.6, ey=-0.8, active=1)
             for _ in range(ndrop)]
    sim = lbm.Sim([p], [phi], [c], [drops], precision=prec, path=lbm.LBM_PATH_WAVE, graph_steps=0)
    lbm.lbm_debug_strips(sim.ctx, lbm.lbm_noalloc_rows(lbm.make_config(p, prec), ndrop))
    nsteps = 3
    got_phi, got_c, at = noalloc(lbm, p, phi, c, sim.droplets(), prec, nsteps)
    sim.step(nsteps)
    want = sim.fields()
    assert np.array_equal(got_phi, want["phi"]) and np.array_equal(got_c, want["c"])
    assert at == [(d["x"], d["y"]) for d in sim.droplets()]
    sim.close()
