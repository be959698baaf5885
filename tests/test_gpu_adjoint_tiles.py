"""The one-launch backward step (tiles) against the three launches, on the same problem.

A lattice and the lattice made of copies of it side by side evolve alike, and the displacement of one droplet has, summed
over the copies, the same derivatives: every copy's field moves with the others'.  The sizes put one of the two on tiles
(at least 21 x 21 nodes, at most 256 tiles of 16 x 16) and the other on the three launches; the smallest tiled height,
ragged last tiles, several droplets, plates.  The two differ by rounding (1e-16 per step and operation of a few hundred;
1e-11 of the largest derivative is allowed for 12 steps)."""
import numpy as np
import pytest

from paper_1711_10984_amd import workloads as W

pytestmark = pytest.mark.gpu


def tiles(nx, ny):
    return nx >= 21 and ny >= 21 and -(-nx // 16) * -(-ny // 16) <= 256


def gradients(nx, ny, walls, copies, prec, path):
    from paper_1711_10984_amd import lbm
    R = min(nx, ny) / 4.0
    drops = [W.DropSpec(x=0.5 * nx + 1.3, y=0.5 * ny - 0.4, R=R, Rs=R / 3.0, ex=0.8, ey=0.6, active=1, psi_front=0.1,
                        psi_back=0.1)]
    phi, c = W.droplet_fields(nx, ny, drops, psi_out=0.1, seed=3)
    p = dict(W.PAPER_EQUILIBRIUM, nx=copies * nx, ny=ny, tau=0.6, gamma=1.5e-3, A0=2e-5, walls=walls)
    table = [dict(x=d.x + k * nx, y=d.y, R=d.R, Rs=d.Rs, ex=d.ex, ey=d.ey, active=1) for d in drops
             for k in range(copies)]
    sim = lbm.Sim([p], [np.tile(phi, (1, copies))], [np.tile(c, (1, copies))], [table], precision=prec, path=path)
    J = sim.adjoint_forward(0, 12, 5)
    dA0, dc0 = sim.adjoint_backward()
    again = sim.adjoint_backward()
    assert again[0] == dA0 and np.array_equal(again[1], dc0)
    sim.close()
    return J, dA0, dc0.reshape(ny, copies, nx).sum(1)


@pytest.mark.parametrize("path", [0, 1, 2])
@pytest.mark.parametrize("nx,ny,copies,walls", [(20, 21, 2, 0), (20, 50, 2, 1), (20, 37, 3, 0), (104, 203, 4, 1)])
def test_one_launch_and_three_give_the_same_derivatives(nx, ny, copies, walls, path):
    assert tiles(nx, ny) != tiles(copies * nx, ny)
    a, b = gradients(nx, ny, walls, 1, 0, path), gradients(nx, ny, walls, copies, 0, path)
    assert abs(a[0] - b[0]) <= 1e-11 * nx
    assert a[1] != 0.0 and abs(a[1] - b[1]) <= 1e-11 * abs(a[1])
    assert np.max(np.abs(a[2] - b[2])) <= 1e-11 * np.max(np.abs(a[2]))


def test_single_precision_agrees_too():
    a, b = gradients(20, 50, 0, 1, 1, 0), gradients(20, 50, 0, 2, 1, 0)
    # FP32 rounds each of a few hundred operations a step at 6e-8
    assert np.max(np.abs(a[2] - b[2])) <= 1e-3 * np.max(np.abs(a[2]))
