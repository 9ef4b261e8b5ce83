"""bench.py names the sweep kernels as the library dispatches them and prices their
bytes by the constants of the header's byte model."""
import os
import re

import pytest

import bench

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.parametrize("wide,form,n,route", [
    (False, 0, 40, "fused"), (False, 1, 41, "streamed"), (False, 0, 64, "streamed"),
    (False, 0, 65, "split"), (False, 1, 400, "split"), (False, 2, 10, "split"),
    (False, -1, 20, "fused"), (False, -1, 21, "packed"), (False, -1, 64, "packed"),
    (False, -1, 65, "split"), (True, 0, 27, "fused"), (True, 0, 28, "streamed"),
    (True, -1, 20, "fused"), (True, -1, 28, "streamed"), (True, 2, 27, "fused"),
    (True, 2, 64, "streamed")])
def test_route(wide, form, n, route):
    assert bench.sweep_route(form, n, wide) == route


def test_bytes_match_the_header():
    text = open(os.path.join(ROOT, "include", "pinmpc.h")).read()
    m = {k: int(v) for k, v in re.findall(r"#define PINMPC_([A-Z]+_BYTES(?:_4)?) (\d+)", text)}
    N = [10, 60]
    for wide, four in ((False, ""), (True, "_4")):
        setup = bench.WIDE_SETUP_BYTES_PER_STAGE if wide else bench.SETUP_BYTES_PER_STAGE
        ops = m["SWEEP_BYTES" + four]
        assert setup + bench.sweep_bytes("fused", 9, N, wide) == m["SETUP_BYTES" + four] + ops
        assert setup + bench.sweep_bytes("streamed", 9, N, wide) == \
            m["SETUP_BYTES" + four] + 9 * ops
    ops, setup = m["SWEEP_BYTES"], bench.SETUP_BYTES_PER_STAGE
    assert setup + bench.sweep_bytes("packed", 9, N, False) == m["SETUP_BYTES"] + 5 * ops
    assert setup + bench.sweep_bytes("split", 9, N, False) == \
        m["SETUP_BYTES"] + 9 * ops + 8 * m["ITERATE_BYTES"]
    assert bench.REFINE_BYTES_PER_PASS_STAGE == m["REFINE_BYTES"]
    assert bench.WIDE_BYTES_PER_IPM_STAGE == m["REFINE_BYTES_4"]
