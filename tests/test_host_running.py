"""lbm_running_kernel and lbm_running_rows name what a step launches, without a GPU."""
import pytest

from hoststub import Context, stubbed

FUSED, SPLIT, WAVE = 0, 1, 2


def launched(lbm, lib, ctx):
    """Names of the kernels that one step launches, among all that the library has for steps."""
    lib.stub_reset()
    lbm.lbm_step(ctx.h, 1)
    mangled = {"k_tile": b"6k_tile", "k_tile_final": b"12k_tile_final", "k_step": b"6k_step", "k_wave": b"6k_wave",
               "k_lb": b"4k_lb", "k_fd": b"4k_fd", "k_reduce": b"8k_reduce"}
    return {k for k, v in mangled.items() if lib.stub_launched(v)}


@pytest.mark.parametrize("nx,tiles", [(64, True), (1200, False)])
def test_names_and_heights_are_those_of_the_step(monkeypatch, nx, tiles):
    lbm, lib = stubbed(monkeypatch)
    ctx = Context(lbm, [(nx, 600 if nx > 64 else 48)], [[dict(x=30.0, y=20.0, R=8.0)]], stream=0)
    names = lambda: {n for n in (lbm.lbm_running_kernel(ctx.h, i) for i in range(3)) if n}
    assert (lbm.lbm_running_kernel(ctx.h, 0) == "k_tile") == tiles and lbm.lbm_running_rows(ctx.h) == (0 if tiles else 64)
    assert names() == launched(lbm, lib, ctx)
    for path, rows in ((SPLIT, 0), (WAVE, 64), (FUSED, 0 if tiles else 64)):
        lbm.lbm_set_path(ctx.h, path)
        assert names() == launched(lbm, lib, ctx) and lbm.lbm_running_rows(ctx.h) == rows
    lbm.lbm_set_seg_rows(ctx.h, 32)
    assert names() == launched(lbm, lib, ctx) == {"k_step", "k_reduce"} and lbm.lbm_running_rows(ctx.h) == 32
    ctx.close()


def test_strips_that_the_autotuner_shortened(monkeypatch):
    """Every launch takes equally long but those of the strips of 10 rows: the autotuner takes them."""
    lbm, lib = stubbed(monkeypatch)
    ctx = Context(lbm, [(54, 6000)], [[dict(x=30.0, y=20.0, R=8.0)]], stream=0)
    lib.stub_fast_grid(600)  # 54 x 6000 in strips of 54 x 10, a multiple of eight
    rows, path, _ = lbm.lbm_autotune(ctx.h, 2)
    lib.stub_fast_grid(0)
    assert rows in lbm.lbm_tune_rows() and lbm.lbm_get_seg_rows(ctx.h) == rows
    assert lbm.lbm_running_rows(ctx.h) == 10
    assert lbm.lbm_running_kernel(ctx.h, 0) == lbm.lbm_kernel_name(path, 0)
    lbm.lbm_step(ctx.h, 1)
    lbm.lbm_set_seg_rows(ctx.h, rows)
    assert lbm.lbm_running_rows(ctx.h) == rows
    ctx.close()


def test_short_strips_that_cut_the_lattice_alike_are_tried_once(monkeypatch):
    """16 rows are one strip of every listed height, and two strips of 8 rows as of 10, 12 and 14."""
    lbm, lib = stubbed(monkeypatch)
    counts = []
    for nx, ny in ((16, 16), (16, 8)):
        ctx = Context(lbm, [(nx, ny)], [[]], stream=0)
        lib.stub_reset()
        lbm.lbm_autotune(ctx.h, 2)
        # two kernels, two passes of one launch and two more for each height
        counts.append(lib.stub_launched(b"6k_step") + lib.stub_launched(b"6k_wave"))
        ctx.close()
    assert counts == [2 * 2 * 3 * 2, 2 * 2 * 3]
