"""$TSSPIN_RESIDENT_FACTORS=0 makes a complex128 state that one workgroup holds form its phase
factors in the kernel, instead of reading ones stored per plan (host-only runtime, no GPU needed)."""
from __future__ import annotations

import pytest

from tests import host_runtime


@pytest.mark.parametrize("n", [1, 5, 9, 12])
def test_switch(tmp_path, n):
    def run(value):
        return host_runtime.run(tmp_path, "resident_factors", n, host_runtime.C128,
                                env={"TSSPIN_RESIDENT_FACTORS": value})
    assert run("1") == {"stored": 1, "runs": 1}
    assert run("0") == {"stored": 0, "runs": 1}
