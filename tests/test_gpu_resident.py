"""States that one workgroup's registers hold, against the oracle: the sizes where the window
layout changes (overlapping windows, less than a wave, the largest of each precision), every
real record kind from registers, several vectors, and a class of chains whose phase tables do
not fit their buffer at once."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from tests import dense_ref as D

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

C128, C64 = torch.complex128, torch.complex64
# complex64: FP32 storage over 3 steps (about 60 layers, as the other parity tests)
TOL = {C128: 1e-10, C64: 1e-5}


def _dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1305_0036_amd import tsspin
    return tsspin


@pytest.mark.parametrize("n,dtype", [(n, d) for n in (4, 6, 7, 9, 11, 13) for d in (C128, C64)] + [(14, C64)])
def test_resident_states_and_records_against_oracle(n, dtype):
    ts = _dev()
    print("[case] resident", n, dtype, flush=True)
    rng = np.random.default_rng(900 + n)
    bonds, fields = D.random_xyz(rng, n, chain=n > 9)
    states = [D.random_state(rng, n) for _ in range(2)]
    H = ts.Hamiltonian(n, bonds, fields)
    if n > 12:
        H.set_tile_bits(ts.TS_C128 if dtype == C128 else ts.TS_C64, n)
    Ho = oracle.Hamiltonian(n, bonds, fields)
    obs = [("norm",), ("mz",), ("sz", n - 1), ("sx", 0), ("sy", n // 2), ("szsz", 0, n - 1)]
    for order in (1, 4):   # order 1: an odd number of layers per step
        x = [torch.from_numpy(s).to(dtype).cuda() for s in states]
        rec = H.evolve(x[0], 0.06, 3, order, record=obs, rec_every=1).cpu().numpy()
        H.evolve(x, 0.06, 2, order)          # both vectors in one launch
        cur = states[0]
        for r in range(4):
            if r:
                cur = oracle.evolve(Ho, cur, 0.06, 1, order)
            ref = [oracle.expect(Ho, cur, *o) for o in obs]
            assert np.abs(rec[r] - ref).max() < TOL[dtype], r
        refs = [oracle.evolve(Ho, cur, 0.06, 2, order), oracle.evolve(Ho, states[1], 0.06, 2, order)]
        for got, ref in zip(x, refs):
            g = got.cpu().numpy().astype(np.complex128)
            assert np.linalg.norm(g - ref) / np.linalg.norm(ref) < TOL[dtype]


def test_resident_batch_in_groups_of_chains():
    # 12 spins: about 400 KB of phase tables per chain, so 3000 chains take two groups
    ts = _dev()
    n, chains = 12, 3000
    print("[case] resident groups", n, chains, flush=True)
    systems = [(n, [(i, i + 1, 1.0, 1.0, 0.5 + c / chains) for i in range(n - 1)],
                np.tile([0.1, 0.2, 0.3 + c / chains], (n, 1))) for c in range(chains)]
    psi = torch.from_numpy(D.random_state(np.random.default_rng(12), n)).cuda()
    B = ts.Batch(systems)
    packed = psi.repeat(chains)
    B.evolve(packed, 0.05, 1, 4)
    B.evolve(packed, 0.05, 1, 4)             # a replay fills the shared buffer anew
    assert B.stats()["capture_failures"] == 0
    for c in (0, 1, 1499, 2500, 2700, 2999):
        x = psi.clone()
        H = ts.Hamiltonian(*systems[c])
        H.evolve(x, 0.05, 1, 4)
        H.evolve(x, 0.05, 1, 4)
        assert torch.equal(x, packed[c << n:(c + 1) << n]), c
