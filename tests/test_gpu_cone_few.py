"""Light-cone sweeps on both sides of the launch-size rule (needs an MI355X).

A launch of at most 256 workgroups takes the variant with two full LDS buffers; more take the
one that leaves room for four waves per SIMD.  Chains and chains with next-nearest bonds (their
phase steps also reach the inner window bits), plain and recorded sweeps, both precisions,
against the ping-pong sweeps of the same library.
"""
from __future__ import annotations

import numpy as np
import pytest

from tests import dense_ref as D

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("dtype", [torch.complex128, torch.complex64])
@pytest.mark.parametrize("nnn", [False, True])
@pytest.mark.parametrize("T,n", [(11, 19), (11, 20), (12, 13), (12, 20), (12, 21)])
def test_both_sides_of_the_launch_size_rule(monkeypatch, T, n, nnn, dtype):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1305_0036_amd import tsspin as ts
    code = ts.TS_C128 if dtype == torch.complex128 else ts.TS_C64
    seed = 5000 + 100 * T + n
    print("[case] few tiles", T, n, nnn, dtype, seed, flush=True)
    rng = np.random.default_rng(seed)
    bonds, fields = D.random_xyz(rng, n, chain=True)
    if nnn:
        bonds = list(bonds) + [(i, i + 2, *rng.uniform(0.2, 0.6, 3)) for i in range(n - 2)]
    g = torch.Generator().manual_seed(seed)
    psi = torch.polar(torch.full((1 << n,), 2.0 ** (-n / 2), dtype=torch.float64),
                      torch.rand(1 << n, dtype=torch.float64, generator=g) * 6.283).to(dtype).cuda()
    out = {}
    for mode in (0, 2):
        monkeypatch.setenv("TSSPIN_CONE", str(mode))
        H = ts.Hamiltonian(n, bonds, fields)
        H.set_tile_bits(code, T)
        if mode == 2:
            assert H.cone_plan(code, 0.03, 2, 4, tile_bits=T)[1]
        x = psi.clone()
        r = H.evolve(x, 0.03, 4, 4, record=[("sz", 1), ("szsz", 0, n - 1), ("norm",)], rec_every=2)
        torch.cuda.synchronize()
        out[mode] = (x.cpu().numpy().astype(np.complex128), r.cpu().numpy())
    err = float(np.linalg.norm(out[2][0] - out[0][0]) / np.linalg.norm(out[0][0]))
    derr = float(np.abs(out[2][1] - out[0][1]).max())
    print("[case]   rel L2", err, "max |drec|", derr, flush=True)
    tol = (1e-11, 1e-12) if dtype == torch.complex128 else (1e-5, 1e-5)
    assert err < tol[0] and derr < tol[1]
