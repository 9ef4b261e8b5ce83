"""GPU kernels at the edges of their dispatch, through the C ABI.

  * refinement by two waves per problem (batches up to 1024) and by one (above)
    give bitwise the same results, at horizons around the rings of the chains
    (multiples of 2, 3, 4, 6 and 12 stages and one beside them), around one
    contact-stage per lane (32 stages) and around the LDS stage buffers (64);
  * those short horizons match the FP64 oracle (the bars of the parity tests),
    also with the normal-force bound active (faces with f_z at its bound);
  * the fused sweep's workgroup sizes for four contacts (13/14, 20/21, 27/28
    stages) and the fused kernel's last horizon for two (40/41): ADMM iterates
    against the FP64 reference at the bars of the iterate tests (one sweep FP32
    rounding 1e-4, three sweeps 1e-3), both forms bitwise equal;
  * stage matrices in blocks of 16 stages, written 16 bytes per lane or, to a
    base that does not allow it, float by float: bitwise the same, and nothing
    outside the outputs written.
"""
import numpy as np
import pytest

import mpcgen
from gpu_common import _check_invariants, _compare, _solve, reset_settings

pytestmark = pytest.mark.gpu

PLAIN, HANDS = "plain_b4096_n20", "hands_b4096_n20"


def _batch(base, horizons, count, n_max, seed):
    cfg = dict(mpcgen.CONFIGS[base], horizons=horizons, batch=count, seed=seed)
    return mpcgen.make_batch(cfg, indices=range(count), n_max=n_max)


@pytest.mark.parametrize("horizons,n_max", [
    ((1, 2, 3, 4, 5), 5), ((6, 7, 11, 12, 13), 13), ((20, 24, 25), 25),
    ((31, 32, 33, 48), 48), ((63, 64), 64), ((64, 65), 65)])
def test_two_waves_and_one_wave_agree_bitwise(solver, horizons, n_max):
    many = _batch(PLAIN, horizons, 1025, n_max, 41)
    few = mpcgen.problem_slice(many, np.arange(1024))
    one, two = _solve(solver, many), _solve(solver, few)
    assert (two["status"] == 0).all()
    for k in two:
        assert np.array_equal(one[k][:1024], two[k]), k


@pytest.mark.parametrize("horizons,fz", [((1, 2, 3, 4, 5, 7), None), ((8, 13), None),
                                         ((6, 12, 13), 0.6)])
def test_short_horizons_match_oracle(solver, horizons, fz):
    batch = _batch(PLAIN, horizons, 24, max(horizons), 42)
    if fz is not None:   # a bound below the weight: f_z at its bound in single stance
        batch["fz_max"] = (fz * batch["mass"] * 9.81).astype(np.float32)
    out = _solve(solver, batch)
    _check_invariants(batch, out, range(24))
    _compare(batch, out, range(24))
    if fz is not None:
        fzs = out["u"][:, :, [2, 8]]
        assert (fzs >= 0.999 * batch["fz_max"][:, None, None]).any()


@pytest.mark.parametrize("horizons", [(1, 2, 3, 4, 5), (8, 9)])
def test_hands_short_horizons_match_oracle(solver, horizons):
    batch = _batch(HANDS, horizons, 20, max(horizons), 43)
    out = _solve(solver, batch, iters=20)
    _check_invariants(batch, out, range(20))
    _compare(batch, out, range(20))


@pytest.mark.parametrize("base,n_max", [(HANDS, 13), (HANDS, 14), (HANDS, 20), (HANDS, 21),
                                        (HANDS, 27), (HANDS, 28), (PLAIN, 40), (PLAIN, 41)])
def test_sweep_iterates_at_workgroup_edges(solver, base, n_max):
    import torch
    from oracle import admm
    from paper_2606_05687_amd import binding
    batch = _batch(base, (n_max, max(1, n_max // 2)), 4, n_max, 44)
    nu = 24 if base == HANDS else 12
    dev = binding.to_device(batch)
    reset_settings(solver)
    for K, tol in ((1, 1e-4), (3, 1e-3)):
        z = {}
        for form in (0, 1):
            solver.set(form=form)
            z[form] = solver.admm(dev, K)
            torch.cuda.synchronize()
            z[form] = z[form].cpu().numpy()
        assert np.array_equal(z[0], z[1])
        for b in range(4):
            p = mpcgen.problem_fp64(batch, b)
            ref = admm.solve(p, iters=K, rho=10.0, scaling=True, accel=True)
            zr = ref["iterates"]["z"].copy()
            zr[:, 13:] *= ref["setup"]["S"]
            scale = np.concatenate([np.ones(13), np.full(nu, p["weight"])])
            zb = z[0][b, :p["N"]].astype(np.float64)
            d = np.max(np.abs(zb - zr) / scale) / max(1.0, np.max(np.abs(zr) / scale))
            assert d <= tol, (K, b, d)


@pytest.mark.parametrize("model", ["srb", "momentum"])
@pytest.mark.parametrize("count,n", [(1, 1), (3, 5), (5, 16), (7, 23)])
def test_stage_matrices_unaligned_outputs(model, count, n):
    import torch
    from paper_2606_05687_amd import binding
    rng = np.random.default_rng([45, count, n])
    phys = dict(
        N=rng.integers(1, n + 1, count).astype(np.int32), yaw_k=rng.normal(0, 2, (count, n)),
        c_ref=rng.normal(0, 1, (count, n, 3)), feet=rng.normal(0, 1, (count, n, 2, 3)),
        mass=rng.uniform(10, 60, count), inertia=rng.uniform(0.1, 3, (count, 3)),
        dt=rng.uniform(0.01, 0.1, count))
    dev = {k: torch.from_numpy(v if k == "N" else v.astype(np.float32)).cuda()
           for k, v in phys.items()}
    sizes, got = (count * n * 169, count * n * 156), []
    for off in (0, 1):
        flat = [torch.full((s + 8,), 7.0, device="cuda") for s in sizes]
        A = flat[0][off:off + sizes[0]].view(count, n, 13, 13)
        B = flat[1][off:off + sizes[1]].view(count, n, 13, 12)
        binding.build_dynamics(dev, A, B, model=model)
        torch.cuda.synchronize()
        for f, s in zip(flat, sizes):
            assert (f[:off] == 7.0).all() and (f[off + s:] == 7.0).all()
        got.append((A.cpu().numpy(), B.cpu().numpy()))
    assert np.array_equal(got[0][0], got[1][0]) and np.array_equal(got[0][1], got[1][1])
    A = got[0][0]
    assert np.array_equal(A[..., np.arange(13), np.arange(13)], np.ones((count, n, 13), np.float32))
