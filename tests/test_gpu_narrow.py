"""Tile widths of small complex128 states (needs an MI355X).

States of 13 to 19 spins in the ping-pong form run on narrow tiles, or (13) on the whole state in
one workgroup; 12 and 20 are the neighbours on either side.  Rings and a fully coupled system, and
chains (light-cone form, windows spread evenly), each order, odd step counts, against the FP64
oracle, and the same call repeated bit for bit.
"""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from tests import dense_ref as D

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("geom", ["chain", "ring", "all"])
@pytest.mark.parametrize("n,order,nsteps", [(12, 4, 2), (13, 4, 3), (14, 1, 3), (14, 4, 2), (15, 2, 3), (16, 4, 1),
                                            (17, 4, 1), (18, 2, 2), (19, 2, 1), (20, 1, 1)])
def test_widths_of_small_states(n, order, nsteps, geom):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1305_0036_amd import tsspin as ts
    seed = 300 * n + 10 * order + nsteps
    print("[case] narrow tiles", n, order, nsteps, geom, seed, flush=True)
    rng = np.random.default_rng(seed)
    bonds, fields = D.random_xyz(rng, n, chain=True)
    if geom == "ring":
        bonds = list(bonds) + [(0, n - 1, 0.7, -0.4, 0.9)]
    elif geom == "all":
        bonds = [(i, j, *rng.uniform(-0.3, 0.3, 3)) for i in range(n) for j in range(i)]
    psi0 = D.random_state(rng, n)
    H = ts.Hamiltonian(n, bonds, fields)
    out = []
    for _ in range(2):
        x = torch.from_numpy(psi0).cuda()
        r = H.evolve(x, 0.05, nsteps, order, record=[("norm",), ("sz", n - 1)])
        torch.cuda.synchronize()
        out.append((x.cpu().numpy(), r.cpu().numpy()))
    assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1])
    ref = oracle.evolve(oracle.Hamiltonian(n, bonds, fields), psi0, 0.05, nsteps, order)
    err = float(np.linalg.norm(out[0][0] - ref) / np.linalg.norm(ref))
    print("[case]   rel L2", err, H.kernel_config(ts.TS_C128, order), flush=True)
    assert err < 1e-10 and abs(out[0][1][-1, 0] - 1.0) < 1e-10
