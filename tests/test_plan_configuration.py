"""A plan belongs to the kernel configuration that it was made under: tuning a context that has
evolved before neither breaks its next call nor keeps the tuner from timing the light-cone form.
On the host-only runtime (no GPU needed)."""
from __future__ import annotations

import json

import pytest

from tests import host_runtime


@pytest.mark.parametrize("dtype", [host_runtime.C128, host_runtime.C64])
def test_call_after_tuning_to_another_register_window(tmp_path, dtype):
    # the cached tuning names the width of the untuned plan with 8 amplitudes per thread, which
    # the light-cone kernel does not have
    cache = tmp_path / "tune.json"
    cache.write_text(json.dumps({"entries": [{"arch": "host", "n": 20, "dtype": dtype, "order": 4, "tile_bits": 12,
                                              "reg_bits": 3, "variant": 0, "ms_per_step": 1.0}]}))
    got = host_runtime.run(tmp_path, "tuned_after_evolving", dtype, env={"TSSPIN_TUNE_CACHE": str(cache)})
    assert got["before"] > 0 and got["after_cone"] == 0 and got["after_reg"] > 0


@pytest.mark.parametrize("dtype", [host_runtime.C128, host_runtime.C64])
def test_tuner_times_the_light_cone_form(tmp_path, dtype):
    got = host_runtime.run(tmp_path, "tuner_launches", dtype, env={"TSSPIN_TUNE_CACHE": str(tmp_path / "t.json")})
    assert got["cone"] > 0
