"""Local energies where a chunk has several times as many entries as the sector
has configurations, and each is found by its place in a map of all of them,
against a plan with the hash tables (chunks of one sample each).

Each row's log psi depends on that row alone, and each sample's sum on its own
entries, so the local energies are equal, bit for bit, where both plans' chunks
go row by row (these networks, of at most 256 units).
"""
import math

import numpy as np
import pytest
import torch

from gen import init_params

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nqs():
    import paper_2208_05637_amd as m
    m.load()
    return m


# (n, n_up, n_dn, precision, flips, conserving flips only, samples): maps of less
# than a tile (4,096 places), one, a few and the largest, an odd number of
# qubits, no sector, a sector of one configuration, entries outside the sector
CASES = [
    (3, -1, -1, "fp64", 6, False, 300),
    (5, 2, 1, "fp64", 14, False, 400),
    (8, 4, 0, "fp64", 40, False, 500),
    (11, 3, 2, "fp32", 120, False, 900),
    (12, 3, 3, "fp64", 60, True, 700),
    (13, -1, -1, "bf16w", 700, False, 300),
    (16, 2, 2, "bf16", 300, True, 500),
    (20, 1, 2, "bf16x3", 150, False, 2500),
    (28, 1, 1, "fp32", 400, False, 90000),
]


def _flip(n, rng, conserving):
    if conserving:   # moves one or two particles within a spin
        q = 2 * rng.choice(n // 2, size=2, replace=False) + int(rng.integers(0, 2))
    else:
        q = rng.choice(n, size=min(n, int(rng.integers(1, 5))), replace=False)
    return sum(1 << int(i) for i in q)


@pytest.mark.parametrize("n,nu,nd,prec,G,cons,B", CASES)
@pytest.mark.parametrize("dedup", [False, True])
def test_sector_index_equals_entries(nqs, n, nu, nd, prec, G, cons, B, dedup):
    print(f"sector index: n={n} sector=({nu},{nd}) {prec} flips={G} B={B} dedup={dedup}", flush=True)
    rng = np.random.default_rng(n * 100 + G)
    flips = {0}
    for _ in range(20 * G):
        if len(flips) <= G:
            flips.add(_flip(n, rng, cons))
    flips = sorted(flips)
    z = [int(rng.integers(0, 2**62)) & ((1 << n) - 1) & ~f for f in flips]      # no Y: real coefficients
    ctx = nqs.Context(0)
    H = nqs.Hamiltonian(n, np.array(flips, dtype=np.uint64), np.array(z, dtype=np.uint64), rng.normal(size=len(flips)),
                        conserves_spin=False).upload(ctx)
    h = {"fp64": 64, "fp32": 128}.get(prec, 256)
    params = torch.from_numpy(init_params(n, 2, h, seed=3)).cuda()
    if nu < 0:
        sector = 1 << n
        x = rng.integers(0, sector, size=B)
    else:
        sector = math.comb((n + 1) // 2, nu) * math.comb(n // 2, nd)
        x = np.zeros(B, dtype=np.int64)
        for i in range(B):
            for q in 2 * rng.permutation((n + 1) // 2)[:nu]:
                x[i] |= 1 << int(q)
            for q in 2 * rng.permutation(n // 2)[:nd] + 1:
                x[i] |= 1 << int(q)
        x[B // 2] = (1 << n) - 1                                               # outside the sector: no amplitude
    assert B * (len(flips) - 1) >= 4 * sector
    x = torch.from_numpy(x.astype(np.int64)).cuda()
    plan = nqs.Plan(ctx, H, 2, h, nu, nd, prec, max_batch=B, dedup=dedup)
    ref = nqs.Plan(ctx, H, 2, h, nu, nd, prec, max_batch=64, dedup=True, chunk_samples=1)
    plan.profile()
    got = nqs.local_energy(plan, params, x)
    rows = plan.profile_read()["forward_rows"]
    assert rows <= B + sector
    some = np.unique(np.concatenate([np.arange(min(B, 40)), [B // 2], rng.integers(0, B, size=20)]))[:64]
    want = nqs.local_energy(ref, params, x[torch.from_numpy(some).cuda()].contiguous())
    assert nqs.device_status(plan) == nqs.device_status(ref)
    np.testing.assert_array_equal(got.cpu().numpy()[some], want.cpu().numpy())
    keep = np.ones(B, dtype=bool)
    if nu >= 0:
        keep[B // 2] = False
    assert np.isfinite(got.cpu().numpy()[keep]).all()
