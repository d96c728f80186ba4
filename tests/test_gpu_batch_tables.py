"""Phase tables of resident batch chains (needs an MI355X): chains that run in groups which fill a
shared buffer in turn, and programs that share a class's tables, give the states and records of one
launch over tables of their own, bit for bit, on first calls and on replays."""
from __future__ import annotations

import numpy as np
import pytest

from tests import dense_ref as D

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

CHAIN = {"complex128": 10 * 2056 * 16, "complex64": 10 * 4096 * 16}   # 12 spins, order 4


def _dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1305_0036_amd import tsspin
    return tsspin


def _systems(n, chains):
    rng = np.random.default_rng(1200 + n)
    return [(n, *D.random_xyz(rng, n, chain=True)) for _ in range(chains)]


@pytest.mark.parametrize("record", [False, True])
@pytest.mark.parametrize("dtype", ["complex128", "complex64"])
def test_groups_against_one_launch(monkeypatch, dtype, record):
    ts = _dev()
    n, chains = 12, 5
    print("[case] groups", dtype, record, flush=True)
    systems = _systems(n, chains)
    psi = torch.from_numpy(D.random_state(np.random.default_rng(3), n)).to(getattr(torch, dtype)).cuda()
    rec = [("sz", 0), ("norm",), ("sx", n - 1)] if record else ()
    out = []
    for limit in (None, 2 * CHAIN[dtype] + 1):   # all five at once; groups of 2, 2 and 1
        if limit is not None:
            monkeypatch.setenv("TSSPIN_RESIDENT_TAB_BYTES", str(limit))
        B = ts.Batch(systems)
        packed, got = psi.repeat(chains), []
        for dt, steps in ((0.05, 2), (0.05, 2), (0.03, 1), (0.05, 2)):   # a first call, replays, another program
            r = B.evolve(packed, dt, steps, 4, record=rec)
            got.append(r.clone() if record else None)
        torch.cuda.synchronize()
        assert B.stats()["capture_failures"] == 0
        out.append((packed, got))
    assert torch.equal(out[0][0], out[1][0])
    if record:
        assert all(torch.equal(a, b) for a, b in zip(out[0][1], out[1][1]))


@pytest.mark.parametrize("dtype", ["complex128", "complex64"])
def test_programs_that_share_tables(dtype):
    ts = _dev()
    n, chains = 9, 7
    print("[case] shared tables", dtype, flush=True)
    B = ts.Batch(_systems(n, chains))
    psi = torch.from_numpy(D.random_state(np.random.default_rng(4), n)).to(getattr(torch, dtype)).cuda()
    states = [psi.repeat(chains) for _ in range(3)]
    streams = [torch.cuda.Stream() for _ in states]
    torch.cuda.synchronize()
    for _ in range(3):
        for x, s in zip(states, streams):   # three programs, at once
            B.evolve(x, 0.04, 5, 4, stream=s)
    torch.cuda.synchronize()
    assert torch.equal(states[0], states[1]) and torch.equal(states[0], states[2])


@pytest.mark.parametrize("dtype", ["complex128", "complex64"])
@pytest.mark.parametrize("n,order", [(3, 4), (5, 2), (9, 1), (10, 4), (12, 4)])
def test_one_chain_of_a_batch_as_alone(n, order, dtype):
    # alone: factors stored ahead, two exchange buffers; in a batch: factors formed in the kernel
    # (complex128) or read where they are used, one buffer
    ts = _dev()
    print("[case] chain alone", n, order, dtype, flush=True)
    rng = np.random.default_rng(500 + n)
    system = (n, *D.random_xyz(rng, n, chain=False))
    psi = torch.from_numpy(D.random_state(rng, n)).to(getattr(torch, dtype)).cuda()
    alone, packed = psi.clone(), psi.clone()
    ts.Hamiltonian(*system).evolve(alone, 0.03, 7, order)
    ts.Batch([system]).evolve(packed, 0.03, 7, order)
    torch.cuda.synchronize()
    assert torch.equal(alone, packed)
