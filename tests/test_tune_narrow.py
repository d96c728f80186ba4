"""Tuning of small complex128 states, whose untuned ping-pong sweeps run on narrow tiles (no GPU
needed): the tuner times that configuration too, and cache entries measured before it are not used."""
from __future__ import annotations

import json

import pytest

from paper_1305_0036_amd import tsspin
from tests import host_runtime


def _entry(n, dtype, **more):
    return {"arch": "none", "n": n, "dtype": dtype, "order": 4, "tile_bits": 12, "reg_bits": 4, "variant": 0,
            "ms_per_step": 0.2, **more}


def _config(n, code):
    bonds = [(i, (i + 1) % n, 1.0, 0.8, 0.6) for i in range(n)]
    return tsspin.Hamiltonian(n, bonds).kernel_config(code, 4)


@pytest.mark.parametrize("n,width", [(14, 9), (15, 9), (16, 10), (19, 11)])
def test_tuner_times_the_untuned_width(tmp_path, n, width):
    got = host_runtime.run(tmp_path, "tuner_widths", n, host_runtime.C128, env={"TSSPIN_TUNE_CACHE": str(tmp_path / "t")})
    assert got["untuned"] == [width, 3] and got["timed"] > 0


@pytest.mark.parametrize("n", [14, 16, 19])
def test_entries_from_before_narrow_widths(tmp_path, monkeypatch, n):
    cache = tmp_path / "tune.json"
    monkeypatch.setenv("TSSPIN_TUNE_CACHE", str(cache))
    monkeypatch.delenv("TSSPIN_NO_TUNE_CACHE", raising=False)
    default = _config(n, tsspin.TS_C128)
    cache.write_text(json.dumps({"entries": [_entry(n, 0), _entry(n, 1), _entry(21, 0)]}))
    assert _config(n, tsspin.TS_C128) == default
    assert _config(n, tsspin.TS_C64)["variant"] == 0      # other sizes and complex64: as measured
    assert _config(21, tsspin.TS_C128)["variant"] == 0
    cache.write_text(json.dumps({"entries": [_entry(n, 0, kernels=2)]}))
    assert _config(n, tsspin.TS_C128) == {"tile_bits": 12, "reg_bits": 4, "variant": 0}
