"""Horizons of at most 64 stages whose interior point passes 40 iterations, from where
the corrector's centring weight has a floor: a normal-force bound little above the
weight and narrow moment bounds, offsets, mixed gaits.  They are certified and match
the oracle, as the long horizons for which the floor was chosen do."""
import numpy as np
import pytest

import mpcgen
from gpu_common import _check_invariants, _compare, _solve

pytestmark = pytest.mark.gpu

SLOW = [28, 39, 393, 539, 761, 1130, 1312, 1437]


@pytest.mark.parametrize("scan", [0, 4])
def test_short_horizons_past_forty_iterations(solver, scan):
    cfg = dict(mpcgen.CONFIGS["uneven_b16384"], horizons=(60,), batch=1500, seed=62)
    batch = mpcgen.make_batch(cfg, indices=SLOW, offsets=True)
    batch["fz_max"] = (1.15 * batch["weight"]).astype(np.float32)
    batch["tau_max"][:] = 2.0
    out = _solve(solver, batch, iters=3, rho=1.0, refine_passes=4, ipm_iters=150,
                 polish_passes=20, scan=scan)
    its = out["detail"][:, 1]
    print("interior-point iterations", its)
    assert (its > 40).sum() >= len(SLOW) // 2 and its.max() < 80
    _check_invariants(batch, out, range(len(SLOW)))
    _compare(batch, out, range(len(SLOW)))
