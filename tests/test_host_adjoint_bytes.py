"""The reverse mode's workspace, without a GPU: what one more step in the interval's record costs."""
from hoststub import Context, stubbed


def test_bytes_of_a_recorded_step(monkeypatch):
    """Ten FP64 stage planes, phi and c (640 columns are whole rows of the pool), and less than a kilobyte beside them."""
    lbm, _ = stubbed(monkeypatch)
    nx, ny = 640, 512
    for precision, field in ((0, 8), (1, 4)):
        ctx = Context(lbm, [(nx, ny)], [[dict(x=9.0, y=8.0, R=5.0)]], precision=precision)
        step = lbm.lbm_adjoint_bytes(ctx.h, 1, 8) - lbm.lbm_adjoint_bytes(ctx.h, 1, 7)
        assert 0 <= step - (10 * 8 + 2 * field) * nx * ny < 1024
        ctx.close()
