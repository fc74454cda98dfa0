"""A chunk between the created chunk and its half, whose ranges of flips by the
usual rule would need more counts than the plan's arrays hold: the same local
energies as in small chunks."""
import numpy as np
import pytest
import torch

from gen import init_params

pytestmark = pytest.mark.gpu

# groups of samples of 256 in the created chunk, in the configured one
CREATED, CHUNK, FLIPS = 179200, 174572, 400


@pytest.mark.parametrize("tables", [False, True])
def test_chunk_between_the_created_one_and_its_half(tables):
    import paper_2208_05637_amd as nqs
    n = 12
    rng = np.random.default_rng(1)
    few = [f for f in range(1, 1 << n) if bin(f).count("1") <= 4]           # (tables take flips of up to four qubits)
    flips = np.sort(rng.choice(few, FLIPS, replace=False)).astype(np.uint64)
    x_mask = np.concatenate([[np.uint64(0)], flips])
    z_mask = np.array([int(rng.integers(0, 1 << n)) & ~int(f) for f in x_mask], dtype=np.uint64)
    ctx = nqs.Context(0)
    H = nqs.Hamiltonian(n, x_mask, z_mask, rng.normal(size=len(x_mask)), conserves_spin=False,
                        **({"tables": True} if tables else {})).upload(ctx)
    params = torch.from_numpy(init_params(n, 1, 64, seed=2)).cuda()
    x = torch.from_numpy(rng.integers(0, 1 << n, CHUNK)).cuda()
    small = nqs.Plan(ctx, H, 1, 64, -1, -1, "fp64", max_batch=CREATED, dedup=False, chunk_samples=4096)
    want = nqs.local_energy(small, params, x)
    del small
    plan = nqs.Plan(ctx, H, 1, 64, -1, -1, "fp64", max_batch=CREATED, dedup=False)
    assert plan.chunk_samples == CREATED
    plan.configure(chunk_samples=CHUNK)
    got = nqs.local_energy(plan, params, x)
    assert nqs.device_status(plan) == 0
    assert torch.equal(got, want)
