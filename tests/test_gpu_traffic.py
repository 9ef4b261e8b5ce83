"""The byte model of pinmpc_stats_traffic on every route of the sweeps: operators
read once where they stay in registers (the default form up to 40 stages, 27 with
four contacts), in every sweep where they are streamed or the horizon is split,
by the problem's horizon class where problems are packed.  Each expected figure is
formed here from the header's constants and the work that the solve reports."""
import os
import re

import numpy as np
import pytest

import mpcgen

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PLAIN, HANDS = "plain_b4096_n20", "hands_b4096_n20"


def _model():
    text = open(os.path.join(ROOT, "include", "pinmpc.h")).read()
    return {k: int(v) for k, v in re.findall(r"#define PINMPC_([A-Z]+_BYTES(?:_4)?) (\d+)", text)}


def _batch(base, n, count=40):
    cfg = dict(mpcgen.CONFIGS[base], horizons=(n, max(1, n // 2)), batch=count, seed=50)
    return mpcgen.make_batch(cfg, indices=range(count), n_max=n)


def _want(batch, out, iters, readings, handed_on=0):
    """readings: operator readings per padded stage (a number or one per problem)."""
    m = _model()
    four = "_4" if batch["B"].shape[-1] == 24 else ""
    n, count = batch["A"].shape[1], batch["A"].shape[0]
    det = out["detail"].cpu().numpy().astype(np.int64)
    passes = int((batch["N"].astype(np.int64) * (det[:, 0] + det[:, 1])).sum())
    reads = int((np.zeros(count, np.int64) + readings).sum()) * n
    return (count * n * m["SETUP_BYTES" + four] + reads * m["SWEEP_BYTES" + four] +
            count * n * handed_on * m["ITERATE_BYTES"] + passes * m["REFINE_BYTES" + four])


@pytest.mark.parametrize("graph", [0, 1])
@pytest.mark.parametrize("base,form,n,iters", [
    (PLAIN, 0, 10, 100), (PLAIN, 1, 40, 5), (PLAIN, 0, 41, 5), (PLAIN, 2, 20, 5),
    (PLAIN, 0, 70, 4), (PLAIN, -1, 20, 3), (PLAIN, -1, 30, 3), (PLAIN, -1, 60, 3),
    (HANDS, 0, 27, 5), (HANDS, -1, 28, 5), (HANDS, 2, 20, 5)])
def test_bytes_follow_the_route(base, form, n, iters, graph):
    import torch
    from paper_2606_05687_amd import binding
    batch = _batch(base, n)
    dev = binding.to_device(batch)
    solver = binding.Solver(0, form=form, iters=iters, graph=graph)
    try:
        out = solver.alloc_out(dev)
        for _ in range(2):                        # the second replays a graph
            solver.solve(dev, out)
        torch.cuda.synchronize()
        tr, ms = solver.traffic(), solver.stats()["total_ms"]
    finally:
        solver.close()
    handed_on = 0
    if base == HANDS:
        readings = 1 if n <= 27 else iters
    elif form == 2 or n > 64:
        readings, handed_on = iters, iters - 1
    elif form == -1 and n > 20:
        readings = np.where(batch["N"] > 40, iters, 1)
    else:
        readings = 1 if n <= 40 else iters
    want = _want(batch, out, iters, readings, handed_on)
    assert tr["bytes"] == pytest.approx(want, rel=1e-12)
    assert tr["gbs"] == pytest.approx(want / (ms * 1e6), rel=1e-3)


def test_replay_after_another_solve():
    """A replayed graph is charged its own shape, not that of the solve before it."""
    import torch
    from paper_2606_05687_amd import binding
    a, b = _batch(PLAIN, 10), _batch(PLAIN, 20, 12)
    da, db = binding.to_device(a), binding.to_device(b)
    solver = binding.Solver(0, iters=7, graph=1)
    try:
        oa, ob = solver.alloc_out(da), solver.alloc_out(db)
        solver.solve(da, oa)
        solver.solve_noalloc(db, ob)
        torch.cuda.synchronize()
        assert solver.traffic()["bytes"] == pytest.approx(_want(b, ob, 7, 1), rel=1e-12)
        solver.solve(da, oa)
        torch.cuda.synchronize()
        assert solver.traffic()["bytes"] == pytest.approx(_want(a, oa, 7, 1), rel=1e-12)
    finally:
        solver.close()
