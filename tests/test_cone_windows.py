"""The windows of complex128 light-cone plans (no GPU needed): spread evenly only where the cost
model finds that cheaper than packed from the left, which is how complex64 plans them."""
from __future__ import annotations

import numpy as np
import pytest

from paper_1305_0036_amd import tsspin


def _bonds(kind, n):
    p = [(i, i + 1) for i in range(n - 1)]
    if kind == "nnn":
        p += [(i, i + 2) for i in range(n - 2)]
    elif kind.startswith("ladder"):
        w = int(kind[-1])
        p = [(i, i + w) for i in range(n - w)] + [(i, i + 1) for i in range(n - 1) if i % w != w - 1]
    return [(i, j, 1.0, 0.8, 0.6) for i, j in p]


def _cost(sweeps, n):
    """The library's model of complex128 sweeps (us)."""
    c = 0.0
    for sw in sweeps:
        layers = sum(bin(op["spins"]).count("1") for op in sw["ops"] if op["kind"] == "bfly")
        phases = sum(op["kind"] == "phase" for op in sw["ops"])
        c += 526.0 + 30.3 * sw["transposes"] + 40.1 * phases + 11.3 * layers
    return c * 2.0 ** (n - 27) + 8.0 * len(sweeps)


@pytest.mark.parametrize("kind,n,order,nsteps,sweeps", [
    ("chain", 23, 4, 4, 25), ("chain", 21, 2, 4, 5), ("chain", 24, 1, 5, 7), ("chain", 25, 1, 5, 7),
    ("chain", 29, 1, 5, 10), ("chain", 30, 1, 5, 10), ("nnn", 23, 2, 4, 9), ("nnn", 26, 4, 1, 15),
    ("nnn", 26, 4, 4, 55), ("nnn", 26, 4, 8, None), ("ladder2", 26, 1, 5, 11), ("ladder3", 24, 1, 5, 12),
    ("ladder3", 25, 4, 4, None), ("ladder3", 26, 4, 1, None)])
def test_windows_never_cost_more_than_packed(kind, n, order, nsteps, sweeps):
    H = tsspin.Hamiltonian(n, _bonds(kind, n), np.full((n, 3), 0.3))
    chosen, _ = H.cone_plan(tsspin.TS_C128, 0.02, nsteps, order, tile_bits=12)
    packed, _ = H.cone_plan(tsspin.TS_C64, 0.02, nsteps, order, tile_bits=12)
    assert _cost(chosen, n) <= _cost(packed, n)
    if sweeps is not None:
        assert len(chosen) == sweeps
