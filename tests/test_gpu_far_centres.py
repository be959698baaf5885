"""Droplets whose centre is far out, infinite or no number: they stay candidates for the nearest centre of a node, so that
no kernel takes an index from an empty list.

Between plates y is not periodic, and a table may hold any finite y: at 1e200 the squared distance overflows.  Such a
droplet, alone, is the nearest of every node, and its sum of phi is that of all nodes with phi >= 0 (N 2^-53 relative for N
nodes; 1e-12 allowed).  Overflowing fields (as in the tests of non-finite tiles) leave centres that are no numbers, here of
as many droplets as a workgroup has threads."""
import numpy as np
import pytest

from paper_1711_10984_amd import workloads as W

pytestmark = pytest.mark.gpu
FUSED, SPLIT, WAVE = 0, 1, 2


def whole_sum(sim):
    phi = sim.fields()["phi"]
    return phi[phi >= 0.0].sum()


@pytest.mark.parametrize("path", [FUSED, SPLIT, WAVE])
@pytest.mark.parametrize("nx,ny,strips", [(64, 48, False), (64, 48, True), (109, 113, True)])
def test_a_far_droplet_is_the_nearest_of_every_node(nx, ny, strips, path):
    from paper_1711_10984_amd import lbm
    f, phi, c = W.random_state(nx, ny, 21)
    p = dict(W.ACTIVE, nx=nx, ny=ny, walls=1)
    sim = lbm.Sim([p], [phi], [c], [[dict(x=20.0, y=1e200, R=8.0, Rs=3.0, active=1)]], f_pre=[f], path=path, graph_steps=0)
    if strips:
        sim.set_seg_rows(16)
    for _ in range(3):
        got, want = sim.observables()["drop_mass"][0], whole_sum(sim)
        assert abs(got - want) <= 1e-12 * want
        sim.step(1)
    sim.close()


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("path", [FUSED, SPLIT, WAVE])
def test_centres_that_are_no_numbers_are_carried_on(path, prec):
    from paper_1711_10984_amd import lbm
    nx, ny, nd = 96, 64, 256
    f, phi, c = W.random_state(nx, ny, 22)
    p = dict(W.ACTIVE, nx=nx, ny=ny, a=-1e6, b=1e6, Gamma=1e306 if prec == 0 else 1e38)
    drops = [dict(x=6.0 * (k % 16) + 2.0, y=4.0 * (k // 16) + 1.5, R=3.0, Rs=1.0, active=k % 2) for k in range(nd)]
    sim = lbm.Sim([p], [phi], [c], [drops], precision=prec, f_pre=[f], path=path, graph_steps=0)
    sim.step(1)
    lost = np.isnan([[d["x"], d["y"]] for d in sim.droplets()]).all(1)
    assert lost.sum() >= 250  # each holds 24 nodes, half of them +inf
    o = sim.observables()
    assert o["nonfinite"] and o["unstable"]
    sim.step(3)
    assert np.isnan([[d["x"], d["y"]] for d in sim.droplets()]).all(1)[lost].all()
    sim.close()
