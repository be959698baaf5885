"""Calls long enough for the tiled step's longer graphs (five graphs' worth of steps): bit for bit the single steps.

By default they are captured by the second call that could use them; lbm_set_graph captures them at once.  Odd remainders
change the starting parity between calls; eager calls and read-backs go between the replays."""
import numpy as np
import pytest

from paper_1711_10984_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("explicit", [False, True])
@pytest.mark.parametrize("nx,ny,walls", [(48, 40, 0), (61, 33, 1)])
def test_long_graphs_equal_single_steps(nx, ny, walls, explicit):
    from paper_1711_10984_amd import lbm
    f, phi, c = W.random_state(nx, ny, 4)
    p = dict(W.ACTIVE, nx=nx, ny=ny, A0=1e-5, tau=0.9, walls=walls)
    drops = [dict(x=0.3 * nx, y=0.5 * ny, R=9.0, Rs=3.0, ex=0.6, ey=0.8, active=1),
             dict(x=0.8 * nx, y=0.4 * ny, R=7.0, Rs=2.0, ex=1.0, ey=0.0, active=1)]
    a = lbm.Sim([p], [phi], [c], [drops], f_pre=[f])
    b = lbm.Sim([p], [phi], [c], [drops], f_pre=[f], graph_steps=0)
    if explicit:
        a.set_graph(4)
    for n in (23, 107, 1, 241, 120):  # 20 to a graph and 100 to a long one (4 and 20)
        a.step(n)
        for _ in range(n):
            b.step(1)
        x, y = a.fields(), b.fields()
        for k in x:
            assert np.array_equal(x[k], y[k]), (n, k)
        assert a.droplets() == b.droplets() and a.step_count == b.step_count
    a.close()
    b.close()
