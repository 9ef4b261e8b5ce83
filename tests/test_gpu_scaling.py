"""Results do not depend on the units of the data, and what is certified is finite.

  * Inputs in another unit (forces and moments divided by s, so B times s and R
    times s^2) pose the same problem: every problem stays certified, after the
    same passes, and the inputs are the same to the parity bars.  The equality
    passes eliminate P H P + (I - P), whose two parts then differ by s^2 in size.
"""
import numpy as np
import pytest

import mpcgen
from gpu_common import TOL_ERR, _check_invariants, _compare, _solve

pytestmark = pytest.mark.gpu

PLAIN, HANDS = "plain_b4096_n20", "hands_b4096_n20"


def _in_units(batch, s):
    out = {k: v.copy() if isinstance(v, np.ndarray) else v for k, v in batch.items()}
    out["B"] *= np.float32(s)
    out["R"] *= np.float32(s) * np.float32(s)
    for k in ("fz_max", "tau_max", "weight", "u_ref", "u_prev"):
        out[k] /= np.float32(s)
    return out


# one wave per problem, two, and the scan; the first passes and the interior point's
# crossover passes
@pytest.mark.parametrize("count,settings", [
    (200, {}), (1100, dict(iters=3, rho=1.0, refine_passes=12, first_passes=0)),
    (96, dict(iters=3, scan=4))])
def test_units_of_the_inputs(solver, count, settings):
    cfg = dict(mpcgen.CONFIGS[PLAIN], horizons=(8, 13, 20), batch=count, seed=47)
    batch = mpcgen.make_batch(cfg, indices=range(count), offsets=True)
    ref = _solve(solver, batch, **settings)
    assert (ref["status"] == 0).all()
    s = 8192.0   # a power of two: the same data, exactly
    out = _solve(solver, _in_units(batch, s), **settings)
    assert (out["status"] == 0).all(), np.flatnonzero(out["status"])
    d = np.abs(out["u"].astype(np.float64) * s - ref["u"]).max((1, 2)) / batch["weight"]
    assert d.max() <= TOL_ERR
    assert np.abs(out["x"].astype(np.float64) - ref["x"]).max() <= TOL_ERR * np.abs(ref["x"]).max()
    assert abs(int(out["iters"].sum()) - int(ref["iters"].sum())) <= 0.01 * int(ref["iters"].sum())


def test_stationarity_with_dominant_input_weights(solver):
    cfg = dict(mpcgen.CONFIGS[PLAIN], horizons=(12,), batch=1000, seed=53)
    batch = mpcgen.make_batch(cfg, indices=range(1000), offsets=True)
    batch["R"] = (batch["R"] * np.float32(1e12)).astype(np.float32)
    out = _solve(solver, batch, ipm_iters=0)
    print("mean r_stat", out["res"][:, 2].mean(), "certified", int((out["status"] == 0).sum()))
    assert out["res"][:, 2].mean() <= 1.1 * 7.1e-10


@pytest.mark.parametrize("base,n,settings", [
    (PLAIN, 20, dict(ipm_iters=0)), (PLAIN, 20, dict(refine_passes=0)),
    (PLAIN, 33, dict(iters=3, scan=4)), (PLAIN, 70, dict(form=2, iters=3)),
    (HANDS, 40, dict(iters=5))])
def test_certified_results_are_finite(solver, base, n, settings):
    cfg = dict(mpcgen.CONFIGS[base], horizons=(n, n // 2), batch=48, seed=48)
    batch = mpcgen.make_batch(cfg, indices=range(48), offsets=True)
    batch["A"] *= np.float32(3.0)
    out = _solve(solver, batch, **settings)
    ok = out["status"] == 0
    finite = np.isfinite(out["u"]).all((1, 2)) & np.isfinite(out["x"]).all((1, 2))
    print("certified", int(ok.sum()), "finite", int(finite.sum()))
    assert finite[ok].all(), np.flatnonzero(ok & ~finite)
    assert (out["res"][ok] <= 1e-9).all()


def test_four_contacts_without_moments(solver):
    cfg = dict(mpcgen.CONFIGS[HANDS], horizons=(5, 13, 20), batch=24, seed=49)
    batch = mpcgen.make_batch(cfg, indices=range(24), offsets=True)
    batch["tau_max"][::2] = 0.0
    out = _solve(solver, batch, iters=10)
    _check_invariants(batch, out, range(24))
    _compare(batch, out, range(24))
    u = out["u"].reshape(24, -1, 4, 6)
    assert np.abs(u[::2, :, :, 3:]).max() <= 1e-6
