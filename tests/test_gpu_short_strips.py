"""Lattices of the sizes where the autotuner may take strips below the listed heights: fields bit for bit those of listed
strips, and the heights that the caller sees unchanged."""
import numpy as np
import pytest

from paper_1711_10984_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [0, 1, 2])
@pytest.mark.parametrize("nx,ny,walls", [(560, 560, 0), (1100, 251, 1), (301, 1009, 0)])
def test_autotuned_strips_give_the_same_fields(nx, ny, walls, prec):
    from paper_1711_10984_amd import lbm
    f, phi, c = W.random_state(nx, ny, 8)
    p = dict(W.ACTIVE, nx=nx, ny=ny, walls=walls, tau=0.9)
    drops = [dict(x=0.4 * nx, y=0.5 * ny, R=40.0, Rs=15.0, ex=0.6, ey=0.8, active=1)]
    a = lbm.Sim([p], [phi], [c], [drops], precision=prec, f_pre=[f])
    b = lbm.Sim([p], [phi], [c], [drops], precision=prec, f_pre=[f], path=lbm.LBM_PATH_WAVE)
    b.set_seg_rows(64)
    rows, path, times = a.autotune(5)
    assert rows == a.seg_rows and rows in a.tune_rows() and path == a.path
    for s in (a, b):
        s.step(25)
    x, y = a.fields(), b.fields()
    for k in x:
        assert np.array_equal(x[k], y[k]), k
    a.set_path(lbm.LBM_PATH_WAVE)
    a.set_seg_rows(rows)  # what it returned can be set
    a.step(2)
    b.step(2)
    assert np.array_equal(a.fields()["phi"], b.fields()["phi"])
    a.close()
    b.close()
