"""A launch that fails in the middle of lbm_step, without a GPU: the steps before it count, and the context says so.

Launch numbers: the strips take two a step (the sweep and the reduction), the split path three, the tiles one a step and
one at the end of the sequence."""
import numpy as np
import pytest

from hoststub import Context, stubbed

DROP = [dict(x=30.0, y=20.0, R=8.0, Rs=3.0, active=1)]
FUSED, SPLIT, WAVE = 0, 1, 2


def context(lbm, path, stream=0):
    ctx = Context(lbm, [(64, 48)], [DROP], stream=stream)  # the null stream: launches one by one
    lbm.lbm_set_path(ctx.h, path)
    return ctx


# (path, launch that fails, steps that stand, kernel of the next step)
CASES = [(FUSED, 0, 0, b"k_tile"), (FUSED, 5, 5, b"k_tile"), (FUSED, 6, 6, b"k_tile"), (WAVE, 6, 3, b"k_wave"),
         (WAVE, 7, 3, b"k_wave"), (SPLIT, 13, 4, b"k_lb"), (SPLIT, 17, 5, b"k_lb")]


@pytest.mark.parametrize("path,first,stand,kernel", CASES)
def test_steps_before_the_failure_count(monkeypatch, path, first, stand, kernel):
    lbm, lib = stubbed(monkeypatch)
    ctx = context(lbm, path)
    lib.stub_reset()
    lib.stub_fail(first, 1)
    with pytest.raises(lbm.LBMError) as e:
        lbm.lbm_step(ctx.h, 10)
    assert e.value.code == lbm.LBM_E_HIP and lbm.lbm_get_step(ctx.h) == stand
    # on tiles the sequence was ended for those steps; the next step starts from their parity
    assert lib.stub_launched(b"k_tile_final") == (path == FUSED and stand > 0)
    lib.stub_reset()
    lib.stub_fail(1, 10)
    with pytest.raises(lbm.LBMError):
        lbm.lbm_step(ctx.h, 1)  # its first kernel alone is launched
    assert lib.stub_launched(kernel) == 1
    lib.stub_reset()
    ctx.close()


@pytest.mark.parametrize("path", [FUSED, WAVE])
@pytest.mark.parametrize("stand", [4, 5])
def test_the_next_step_reads_the_state_that_stands(monkeypatch, path, stand):
    lbm, lib = stubbed(monkeypatch)
    ctx = context(lbm, path)
    lib.stub_reset()
    lib.stub_fail(stand if path == FUSED else 2 * stand, 1)
    with pytest.raises(lbm.LBMError):
        lbm.lbm_step(ctx.h, 10)
    parity = []
    for _ in range(2):
        # one launch of the step's kernel from the current state
        lbm.lbm_debug_stage(ctx.h, 0, np.empty((lbm.LBM_NSTAGE, 48, 64)))
        parity.append(lib.stub_last_int())
        lbm.lbm_step(ctx.h, 1)
    assert parity == [stand % 2, 1 - stand % 2] and lbm.lbm_get_step(ctx.h) == stand + 2
    ctx.close()


def test_a_sequence_of_tiled_steps_that_cannot_be_ended(monkeypatch):
    """Nothing was overwritten after one step; after more the fields and the table belong to different steps."""
    lbm, lib = stubbed(monkeypatch)
    one, many = context(lbm, FUSED), context(lbm, FUSED)
    lib.stub_reset()
    lib.stub_fail(1, 1)
    with pytest.raises(lbm.LBMError):
        lbm.lbm_step(one.h, 1)
    assert lbm.lbm_get_step(one.h) == 0
    lbm.lbm_step(one.h, 3)
    assert lbm.lbm_get_step(one.h) == 3
    lib.stub_reset()
    lib.stub_fail(4, 2)
    with pytest.raises(lbm.LBMError) as e:
        lbm.lbm_step(many.h, 10)
    assert e.value.code == lbm.LBM_E_HIP
    for call in (lambda: lbm.lbm_step(many.h, 1), lambda: many.centres()):
        with pytest.raises(lbm.LBMError) as e:
            call()
        assert e.value.code == lbm.LBM_E_STATE
    one.close()
    many.close()


def test_a_capture_that_fails_changes_nothing(monkeypatch):
    lbm, lib = stubbed(monkeypatch)
    ctx = context(lbm, FUSED, stream=1)
    lib.stub_reset()
    lib.stub_fail(7, 30)
    with pytest.raises(lbm.LBMError):
        lbm.lbm_step(ctx.h, 20)
    lib.stub_reset()
    assert lbm.lbm_get_step(ctx.h) == 0 and ctx.centres() == [(30.0, 20.0)]
    lbm.lbm_step(ctx.h, 20)
    assert lbm.lbm_get_step(ctx.h) == 20
    ctx.close()
