"""Systems on streams of their own run beside each other (needs an MI355X): the light-cone launches
of one leave room on the CUs for the others', and each gets the result that it gets alone."""
from __future__ import annotations

import time

import numpy as np
import pytest

from tests import dense_ref as D

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


# bound: the time of all streams over that of one, the best of several choices of streams (two that
# share a hardware queue run one after the other).  The kernel of four workgroups per CU measured
# 1.24 and 1.73; one that fills the CU with one (complex128) or two workgroups 1.97 and 2.30.
@pytest.mark.parametrize("dtype,streams,bound", [("complex128", 2, 1.6), ("complex64", 4, 2.0)])
def test_light_cone_launches_share_the_cus(dtype, streams, bound):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1305_0036_amd import tsspin as ts
    n = 20
    print("[case] streams", n, dtype, streams, flush=True)
    rng = np.random.default_rng(41)
    psi0 = torch.from_numpy(D.random_state(rng, n)).to(getattr(torch, dtype)).cuda()
    systems = [ts.Hamiltonian(n, *D.random_xyz(rng, n, chain=True)) for _ in range(streams)]
    pool = [torch.cuda.Stream() for _ in range(8)]
    alone = []
    for H in systems:
        x = psi0.clone()
        H.evolve(x, 0.02, 8, 4)
        alone.append(x)
    x = [psi0.clone() for _ in systems]
    torch.cuda.synchronize()

    def timed(own):
        t0 = time.perf_counter()
        for H, y, s in zip(systems, x, own):
            H.evolve(y, 0.02, 8, 4, stream=s)
        torch.cuda.synchronize()
        return time.perf_counter() - t0

    timed(pool[:streams])
    assert all(torch.equal(a, b) for a, b in zip(alone, x))
    one = min(timed(pool[:1]) for _ in range(5))
    many = min(timed(pool[k:k + streams]) for k in range(len(pool) - streams + 1) for _ in range(4))
    print(f"[case]   one {one * 1e6:.0f} us, {streams} at once {many * 1e6:.0f} us", flush=True)
    assert many < bound * one
