"""The strip heights that lbm_step_noalloc chooses: fields bit for bit those of lbm_step at another height.

The sizes: the last lattice with the fixed height and the first with the rule's, odd ones with a remainder of a strip in
x and y, a set of strips that does not divide by eight, one round of wavefronts nearly full, and one of several rounds
(whose strips are listed in natural order).  The centres' sums are rounded strip by strip, at most N 2^-53 relative for
N nodes, so centres agree within 1e-12 of the lattice."""
import numpy as np
import pytest

from paper_1711_10984_amd import workloads as W

MANY = 100  # droplets: the short strips' partials then exceed the scratch array, and strips of 40 rows take the lattice

pytestmark = pytest.mark.gpu
WT = [4 / 9] + [1 / 9] * 4 + [1 / 36] * 4


def noalloc(lbm, p, phi0, c0, drops, prec, nsteps):
    import torch
    dev = torch.device("cuda:0")
    dt = torch.float64 if prec == 0 else torch.float32
    ft = torch.float16 if prec == 2 else dt
    ny, nx = phi0.shape
    f = [torch.zeros((9, ny, nx), dtype=ft, device=dev) for _ in range(2)]
    if prec == 0:
        for i in range(9):
            f[0][i] = WT[i]
    else:
        for i in range(9):
            f[0][i] = float(WT[i] - float(np.float32(WT[i]))) if prec == 1 else 0.0
    phi = [torch.from_numpy(phi0).to(dev, dt), torch.zeros((ny, nx), dtype=dt, device=dev)]
    c = [torch.from_numpy(c0).to(dev, dt), torch.zeros((ny, nx), dtype=dt, device=dev)]
    table = (lbm.lbm_droplet * len(drops))(*[lbm.make_droplet(d) for d in drops])
    dd = torch.from_numpy(np.frombuffer(bytes(table), dtype=np.uint8).copy()).to(dev)
    rc = lbm.lbm_step_noalloc(lbm.make_config(p, prec), torch.cuda.current_stream().cuda_stream,
                              [t.data_ptr() for t in f], [t.data_ptr() for t in phi], [t.data_ptr() for t in c],
                              len(drops), dd.data_ptr(), 0, nsteps)
    assert rc == lbm.LBM_OK, lbm.lbm_last_error()
    torch.cuda.synchronize()
    k = nsteps % 2
    out = (lbm.lbm_droplet * len(drops)).from_buffer_copy(dd.cpu().numpy().tobytes())
    return phi[k].double().cpu().numpy(), c[k].double().cpu().numpy(), [(d.x, d.y) for d in out]


SIZES = [(255, 256, 0), (256, 256, 0), (271, 257, 1), (700, 333, 0), (1000, 1100, 1)]


@pytest.mark.parametrize("nx,ny,walls,prec,ndrop", [s + (p, 5) for s in SIZES for p in (0, 1, 2)] +
                         [(34560, 208, 0, 0, 5), (34560, 208, 0, 0, MANY), (34560, 208, 0, 1, MANY), (57456, 208, 0, 1, 5)])
def test_fields_do_not_depend_on_the_height(nx, ny, walls, prec, ndrop):
    from paper_1711_10984_amd import lbm
    rng = np.random.default_rng(nx + ny)
    p = dict(W.ACTIVE, nx=nx, ny=ny, walls=walls, tau=0.9)
    phi = 0.3 * rng.standard_normal((ny, nx)) - 0.3
    c = 0.05 + 0.01 * rng.standard_normal((ny, nx))
    drops = [dict(x=rng.uniform(0, nx), y=rng.uniform(0, ny), R=ny / 4.0, Rs=ny / 9.0, ex=0.6, ey=-0.8, active=1)
             for _ in range(ndrop)]
    nsteps = 5
    sim = lbm.Sim([p], [phi], [c], [drops], precision=prec, path=lbm.LBM_PATH_WAVE, graph_steps=0)
    sim.set_seg_rows(64)
    got_phi, got_c, at = noalloc(lbm, p, phi, c, sim.droplets(), prec, nsteps)
    sim.step(nsteps)
    want = sim.fields()
    assert np.array_equal(got_phi, want["phi"]) and np.array_equal(got_c, want["c"])
    for q, d in zip(at, sim.droplets()):
        assert abs(q[0] - d["x"]) < 1e-12 * nx and abs(q[1] - d["y"]) < 1e-12 * nx
    sim.close()
