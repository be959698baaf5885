"""The graphs that lbm_set_graph and lbm_step capture, without a GPU: what a caller asks for and no more."""
from hoststub import Context, stubbed


def tiled_context(lbm):
    return Context(lbm, [(64, 48)], [[dict(x=30.0, y=20.0, R=8.0, Rs=3.0, active=1)]])


def test_set_graph_captures_two_graphs_of_its_size(monkeypatch):
    lbm, lib = stubbed(monkeypatch)
    ctx = tiled_context(lbm)
    for n in (2, 20, 300):
        lib.stub_reset()
        lbm.lbm_set_graph(ctx.h, n)
        assert lib.stub_launched(b"k_tile") == 2 * n + 2  # each ends with the kernel that brings the table up to date
    lib.stub_reset()
    for _ in range(3):
        lbm.lbm_step(ctx.h, 1800)
    assert lib.stub_launched(b"k_") == 0  # replays alone
    ctx.close()


def test_default_graphs_of_long_calls_wait_for_the_second_one(monkeypatch):
    lbm, lib = stubbed(monkeypatch)
    ctx = tiled_context(lbm)
    captured = []
    for n in (100, 100, 200, 60):
        lib.stub_reset()
        lbm.lbm_step(ctx.h, n)
        captured.append(lib.stub_launched(b"6k_tile"))
    assert captured == [20, 100, 0, 0]
    assert lbm.lbm_get_step(ctx.h) == 460
    ctx.close()


def test_long_rows_of_single_launches_go_in_sequences(monkeypatch):
    """A tiled step counts the steps before it in its sequence in 32 bits: a sequence ends after 2^20 steps."""
    lbm, lib = stubbed(monkeypatch)
    ctx = Context(lbm, [(64, 48)], [[dict(x=30.0, y=20.0, R=8.0, Rs=3.0, active=1)]], stream=0)
    lib.stub_reset()
    n = (1 << 20) + 3
    lbm.lbm_step(ctx.h, n)
    assert lib.stub_launched(b"6k_tile") == n and lib.stub_launched(b"k_tile_final") == 2
    assert lbm.lbm_get_step(ctx.h) == n
    ctx.close()
