"""The reverse mode in a workspace at any address: the header asks for no alignment, and the gradients do not depend on it.

At an offset that is no multiple of the element size, planes counted in elements from the context's own pool would lie
beside the bytes that were written.  200 x 120 takes the tiled kernels, 560 x 96 strips and three launches."""
import numpy as np
import pytest

from paper_1711_10984_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("nx,ny,path", [(200, 120, 0), (560, 96, 2)])
def test_gradients_do_not_depend_on_the_address(nx, ny, path, prec):
    import torch
    from paper_1711_10984_amd import lbm
    f, phi, c = W.random_state(nx, ny, 11)
    p = dict(W.ACTIVE, nx=nx, ny=ny, A0=1e-6, tau=0.9)
    drops = [dict(x=0.4 * nx, y=0.5 * ny, R=20.0, Rs=7.0, ex=0.8, ey=0.6, active=1)]
    got = {}
    for offset in (0, 4, 2, 129):
        sim = lbm.Sim([p], [phi], [c], [drops], precision=prec, f_pre=[f], path=path, graph_steps=0)
        nbytes = lbm.lbm_adjoint_bytes(sim.ctx, 7, 3)
        ws = torch.zeros(nbytes + offset, dtype=torch.uint8, device="cuda:0")
        J = lbm.lbm_adjoint_forward(sim.ctx, ws.data_ptr() + offset, nbytes, 0, 7, 3)
        got[offset] = (J,) + lbm.lbm_adjoint_backward(sim.ctx, ws.data_ptr() + offset, nbytes, (ny, nx))
        sim.close()
    J, dA0, dc0 = got[0]
    assert dA0 != 0.0 and np.any(dc0)
    for offset in (4, 2, 129):
        assert got[offset][:2] == (J, dA0) and np.array_equal(got[offset][2], dc0), offset
