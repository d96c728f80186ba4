"""Device memory of a batch's phase tables, on the host-only runtime (no GPU needed): programs of
the same steps share them, all programs together keep at most 4 GiB and their groups, and a device
without room for a class's tables makes the groups smaller, not the call fail.  A refused allocation
is not reported by the next call's launches."""
from __future__ import annotations

import pytest

from tests import host_runtime

GIB = 1 << 30
CHAIN = {host_runtime.C128: 10 * 2056 * 16, host_runtime.C64: 10 * 4096 * 16}   # 12 spins, order 4


@pytest.mark.parametrize("dtype", [host_runtime.C128, host_runtime.C64])
def test_programs_of_the_same_steps_share_tables(tmp_path, dtype):
    held = host_runtime.run(tmp_path, "batch_tables", 12, 200, dtype, [0.05], [4096, 8192, 12288])
    tables = 200 * CHAIN[dtype]
    assert held[0] > tables
    assert held[2] - held[0] < tables // 10


def test_tables_of_all_programs_are_bounded(tmp_path):
    # eight time steps (the most programs a batch keeps) of 1.05 GB each
    held = host_runtime.run(tmp_path, "batch_tables", 12, 1600, host_runtime.C64, [0.01 * k for k in range(1, 9)], [4096])
    assert max(held) < 4 * GIB + 5 * (GIB // 4) + GIB // 4


@pytest.mark.parametrize("dtype", [host_runtime.C128, host_runtime.C64])
def test_groups_of_chains(tmp_path, dtype):
    # room for two chains: five chains in groups of 2, 2 and 1, each filled before it runs
    env = {"TSSPIN_RESIDENT_TAB_BYTES": str(2 * CHAIN[dtype] + 1)}
    assert host_runtime.run(tmp_path, "batch_groups", 12, 5, dtype, env=env) == {"fills": 3, "runs": 3}
    assert host_runtime.run(tmp_path, "batch_groups", 12, 5, dtype) == {"fills": 1, "runs": 1}


@pytest.mark.parametrize("dtype", [host_runtime.C128, host_runtime.C64])
def test_short_of_memory(tmp_path, dtype):
    got = host_runtime.run(tmp_path, "batch_short_of_memory", 12, 200, dtype, 100 * CHAIN[dtype])
    assert got["rc"] == 0 and got["failed"] > 0


@pytest.mark.parametrize("dtype", [host_runtime.C128, host_runtime.C64])
@pytest.mark.parametrize("n", [5, 16, 20])
def test_call_after_a_refused_allocation(tmp_path, n, dtype):
    assert host_runtime.run(tmp_path, "call_after_a_refused_allocation", n, dtype) == [-2, 0]
