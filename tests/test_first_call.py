"""What the first call of a new Hamiltonian asks of the device, on the host-only runtime (no GPU
needed): a light-cone plan's phase tables, some hundred, go up in a few buffers, and a system that
stays in the ping-pong form is planned in the light-cone form once."""
from __future__ import annotations

import pytest

from tests import host_runtime


# (eight complex64 steps at 24 spins run in the ping-pong form)
@pytest.mark.parametrize("n,steps,dtype", [(n, s, d) for d in (host_runtime.C128, host_runtime.C64)
                                           for n, s in ((20, 1), (23, 1), (23, 8))] + [(24, 8, host_runtime.C128)])
def test_light_cone_tables_go_up_together(tmp_path, n, steps, dtype):
    got = host_runtime.run(tmp_path, "first_call", n, dtype, steps)
    assert got["sweeps"] > 0
    # 76 to 275 tables of 21 KB (with three or four workgroup rows), a megabyte at a time, and the
    # sweeps' arguments
    assert got["allocs"] <= 8 and got["uploads"] <= 8


@pytest.mark.parametrize("n", [18, 19])
def test_narrow_width_is_planned_once(tmp_path, n):
    # both plan the light-cone form at width 12 and turn it down; planning it again at the narrow
    # width (11, which that form also has) made 1.4 and 1.6 of this (planned once: 0.9 and 1.05)
    assert host_runtime.run(tmp_path, "narrow_first_call", n)["ratio"] < 1.25
