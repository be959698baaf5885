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
    assert rows(70200, 208, 1, 5) == 16 and rows(70200, 208, 1, 60) == 40
    assert rows(4096, 4096, 1, 8) == 16 and rows(4096, 4096, 1, 64) == 40


def test_fixed_heights_where_the_strips_make_many_rounds():
    """5.5 rounds of 3 x 1024 wavefronts in FP32 and of 0.9 x 2 x 1024 in FP64, in strips of 54 x 16."""
    for prec, wavefronts, fixed in ((0, 1843.2, 40), (1, 3072, 16)):
        for n in range(2200, 4400, 37):
            rounds = -(-n // 54) * -(-n // 16) / wavefronts
            assert (rows(n, n, prec, 1) == fixed) == (rounds >= 5.5), (prec, n)


def test_what_is_refused():
    for call, code in ((lambda: rows(8192, 8192, ndrop=256), lbm.LBM_E_NOMEM), (lambda: rows(64, 64, tau=0.4), lbm.LBM_E_INVAL),
                       (lambda: rows(64, 64, ndrop=257), lbm.LBM_E_INVAL), (lambda: rows(2, 64), lbm.LBM_E_INVAL)):
        with pytest.raises(lbm.LBMError) as e:
            call()
        assert e.value.code == code
