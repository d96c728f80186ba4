"""complex64 light-cone sweeps whose phase steps reach the inner bits of the register window
(next-nearest bonds; needs an MI355X): the same states in launches of few and of many workgroups'
kernels as complex128 to FP32 rounding, and no dearer against a chain than the products ask."""
from __future__ import annotations

import time

import numpy as np
import pytest

from tests import dense_ref as D

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _systems(ts, n):
    rng = np.random.default_rng(70 + n)
    bonds, fields = D.random_xyz(rng, n, chain=True)
    nnn = list(bonds) + [(i, i + 2, *rng.uniform(0.2, 0.6, 3)) for i in range(n - 2)]
    return ts.Hamiltonian(n, bonds, fields), ts.Hamiltonian(n, nnn, fields)


def _state(n, dtype):
    g = torch.Generator(device="cuda").manual_seed(n)
    return torch.polar(torch.full((1 << n,), 2.0 ** (-n / 2), dtype=torch.float64, device="cuda"),
                       torch.rand(1 << n, dtype=torch.float64, device="cuda", generator=g) * 6.283).to(dtype)


@pytest.mark.parametrize("n", [19, 20, 21])
def test_inner_window_bits_against_complex128(n):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1305_0036_amd import tsspin as ts
    print("[case] masks", n, flush=True)
    for H in _systems(ts, n):
        assert H.cone_plan(ts.TS_C64, 0.03, 2, 4)[1]
        a, b = _state(n, torch.complex64), _state(n, torch.complex64).to(torch.complex128)
        H.evolve(a, 0.03, 2, 4)
        H.evolve(b, 0.03, 2, 4)
        assert float((a.to(torch.complex128) - b).norm() / b.norm()) < 1e-5


def test_inner_window_bits_cost_their_products():
    # a step with next-nearest bonds against one of the chain, 2^26 amplitudes: 1.21 with the
    # window's factors held, 1.41 with each loaded again where it is used
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1305_0036_amd import tsspin as ts
    n = 26
    print("[case] masks, time", n, flush=True)
    x = _state(n, torch.complex64)
    t = []
    for H in _systems(ts, n):
        H.evolve(x, 0.02, 1, 4)
        torch.cuda.synchronize()
        reps = []
        for _ in range(6):
            t0 = time.perf_counter()
            H.evolve(x, 0.02, 1, 4)
            torch.cuda.synchronize()
            reps.append(time.perf_counter() - t0)
        t.append(min(reps))
    print(f"[case]   chain {t[0] * 1e3:.2f} ms, next-nearest {t[1] * 1e3:.2f} ms", flush=True)
    assert t[1] < 1.3 * t[0]
