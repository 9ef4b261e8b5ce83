"""The sweep kernels against each other, forced apart by padding.

One launch holds all sweeps either way (forms 0 and 1), and the padded horizon
alone decides between the kernel that keeps a problem's operators in registers
(up to 27 stages with four contacts, 40 with two) and the one that streams
them.  The same problems padded to one stage more run the other kernel, and
their iterates have to be bitwise the same: after one sweep, a few, and enough
for restarts of the acceleration (whose decisions compare sums of squares, so
one different rounding shows), with FP32 and BF16 operators.
"""
import numpy as np
import pytest

import mpcgen
from gpu_common import reset_settings

pytestmark = pytest.mark.gpu

PLAIN, HANDS = "plain_b4096_n20", "hands_b4096_n20"
COUNT = 7


def _iterates(solver, base, n, n_max, sweeps, **settings):
    import torch
    from paper_2606_05687_amd import binding
    cfg = dict(mpcgen.CONFIGS[base], horizons=(n, max(1, n // 2)), batch=COUNT, seed=46)
    batch = mpcgen.make_batch(cfg, indices=range(COUNT), n_max=n, offsets=True)
    assert batch["N"].max() == n
    for k in ("A", "B", "e", "x_ref", "u_ref", "contact"):
        pad = [(0, 0)] * batch[k].ndim
        pad[1] = (0, n_max - n)
        batch[k] = np.pad(batch[k], pad)
    reset_settings(solver)
    solver.set(**settings)
    z = solver.admm(binding.to_device(batch), sweeps)
    torch.cuda.synchronize()
    z = z.cpu().numpy()
    return [z[b, :batch["N"][b]] for b in range(COUNT)]


# the workgroup bounds of the register kernel with four contacts (512, 768 and
# 1024 threads), against the streaming kernel at two and three rows a thread
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("n,streamed", [(13, 28), (20, 28), (21, 56), (27, 28), (27, 64)])
def test_four_contacts_registers_equal_streamed(solver, n, streamed, precision):
    for sweeps in (1, 3, 37, 100):
        a = _iterates(solver, HANDS, n, n, sweeps, precision=precision)
        b = _iterates(solver, HANDS, n, streamed, sweeps, precision=precision)
        assert all(np.array_equal(x, y) for x, y in zip(a, b)), sweeps
        assert all(np.isfinite(x).all() for x in a)


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("n,group", [(10, 1), (10, 2), (10, 4), (20, 1), (20, 2), (40, 1)])
def test_two_contacts_registers_equal_streamed(solver, n, group, precision):
    for sweeps in (1, 37, 100):
        a = _iterates(solver, PLAIN, n, n, sweeps, precision=precision, group=group)
        b = _iterates(solver, PLAIN, n, 41, sweeps, precision=precision)
        assert all(np.array_equal(x, y) for x, y in zip(a, b)), sweeps


@pytest.mark.parametrize("base,n,streamed", [(HANDS, 27, 28), (PLAIN, 40, 41)])
def test_without_acceleration(solver, base, n, streamed):
    a = _iterates(solver, base, n, n, 20, accel=0)
    b = _iterates(solver, base, n, streamed, 20, accel=0)
    assert all(np.array_equal(x, y) for x, y in zip(a, b))


# the builds of the register kernel, with and without spilled registers: chosen by
# how many workgroups a CU gets (up to 512 threads per workgroup)
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("n,group,many", [(5, 1, 1100), (5, 2, 1100), (5, 4, 1100),
                                          (10, 1, 600), (10, 2, 600), (20, 1, 300)])
def test_few_and_many_problems_agree_bitwise(solver, n, group, many, precision):
    import torch
    from paper_2606_05687_amd import binding
    cfg = dict(mpcgen.CONFIGS[PLAIN], horizons=(n, max(1, n // 2)), batch=COUNT, seed=51)
    few = mpcgen.make_batch(cfg, indices=range(COUNT), n_max=n, offsets=True)
    rep = np.arange(many) % COUNT
    z = []
    for batch in (few, mpcgen.problem_slice(few, rep)):
        reset_settings(solver)
        solver.set(group=group, precision=precision)
        z.append([solver.admm(binding.to_device(batch), k) for k in (3, 20, 50)])
        torch.cuda.synchronize()
        z[-1] = [v.cpu().numpy() for v in z[-1]]
    for a, b in zip(*z):
        for i in range(COUNT):
            k = few["N"][i]
            assert (b[rep == i][:, :k] == a[i, :k]).all()
