"""The strip height of lbm_step_noalloc, without a GPU: its range, the lattices that keep 40 rows, and what is refused."""
import random

import pytest

from paper_1711_10984_amd import lbm


def rows(nx, ny, prec=0, ndrop=5, **kw):
    return lbm.lbm_noalloc_rows(lbm.make_config(dict(nx=nx, ny=ny, **kw), prec), ndrop)


def test_range():
    rng = random.Random(5)
    for _ in range(300):
        nx, ny = (int(3 * 1000 ** rng.random()) for _ in range(2))
        h = rows(nx, ny, rng.randrange(3))
        assert 4 <= h <= 128 and (nx * ny >= 256 * 256 or h == 40)


def test_forty_rows_where_short_strips_exceed_the_scratch_array():
    assert rows(57456, 208, 1, 5) == 16 and rows(57456, 208, 1, 100) == 40
    assert rows(4096, 4096, 1, 8) == 16 and rows(4096, 4096, 1, 64) == 40


def test_what_is_refused():
    for call, code in ((lambda: rows(8192, 8192, ndrop=256), lbm.LBM_E_NOMEM), (lambda: rows(64, 64, tau=0.4), lbm.LBM_E_INVAL),
                       (lambda: rows(64, 64, ndrop=257), lbm.LBM_E_INVAL), (lambda: rows(2, 64), lbm.LBM_E_INVAL)):
        with pytest.raises(lbm.LBMError) as e:
            call()
        assert e.value.code == code
