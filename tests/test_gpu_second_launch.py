"""The refinement's second launch runs its problems by two waves each or, where the
first leaves it many (few active-set passes there, or none), by one: bitwise the same
results either way, in horizons up to 64 stages and beyond."""
import numpy as np
import pytest

import mpcgen
from gpu_common import _solve

pytestmark = pytest.mark.gpu

COUNT, MANY = 30, 2700   # 2700: more than 2.5 problems per SIMD of the whole chip


@pytest.mark.parametrize("horizons,settings", [
    ((1, 4, 7, 12), dict(refine_passes=0)), ((5, 13), dict(iters=3, first_passes=1)),
    ((20, 33), dict(iters=3, first_passes=1)), ((65,), dict(iters=3, refine_passes=0))])
def test_many_listed_problems(solver, horizons, settings):
    cfg = dict(mpcgen.CONFIGS["plain_b4096_n20"], horizons=horizons, batch=COUNT, seed=52)
    few = mpcgen.make_batch(cfg, indices=range(COUNT), n_max=max(horizons), offsets=True)
    rep = np.arange(MANY) % COUNT
    a = _solve(solver, few, **settings)
    b = _solve(solver, mpcgen.problem_slice(few, rep), **settings)
    assert (a["status"] == 0).all()
    if "refine_passes" in settings:
        assert (b["detail"][:, 3] == 2).sum() > 2560
    for k in a:
        assert np.array_equal(b[k], a[k][rep]), k
