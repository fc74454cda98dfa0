"""Gradient sums over three and more blocks of samples: with room for all blocks'
sums, for some at a time, and for none (one workgroup takes the blocks in turn) the
same bits.  The room is the dead part of the plan's workspace, which grows with
its chunk."""
import numpy as np
import pytest
import torch

from gen import init_params

pytestmark = pytest.mark.gpu

# (precision, width, samples): blocks of 256 samples (FP64 64); a hidden layer's sums of one block take h^2 values,
# where the workspace has 340 bytes of room per sample of the chunk
CASES = [("fp32", 512, 600), ("fp32", 512, 1025), ("bf16w", 512, 777), ("fp64", 256, 600), ("fp64", 256, 193)]


@pytest.mark.parametrize("prec,h,B", CASES)
def test_block_sums_do_not_depend_on_the_room(prec, h, B):
    import paper_2208_05637_amd as nqs
    n, L = 20, 2
    rng = np.random.default_rng(3)
    f = np.array([0, 3, 12], dtype=np.uint64)
    ctx = nqs.Context(0)
    H = nqs.Hamiltonian(n, f, np.zeros(3, dtype=np.uint64), np.array([0.3, -0.7, 0.4]), conserves_spin=False).upload(ctx)
    params = torch.from_numpy(init_params(n, L, h, seed=2)).cuda()
    x = torch.from_numpy(rng.choice(1 << n, B, replace=False)).cuda()
    w = torch.from_numpy(rng.integers(1, 50, B).astype(np.float64)).cuda()
    got = []
    per = h * h * (8 if prec == "fp64" else 4)
    for batch in (B, 8000, 60000):
        plan = nqs.Plan(ctx, H, L, h, -1, -1, prec, max_batch=batch, dedup=False)
        room = batch * (8 * 32 + 16 + 2 * 32)                  # partial sums, diagonal, entries
        print(f"{prec} h={h} B={B}: room for about {room / per:.1f} of {-(-B // (64 if prec == 'fp64' else 256))} "
              f"blocks", flush=True)
        _, grad, _ = nqs.energy_grad(plan, params, x, w)
        got.append(grad)
    assert bool(torch.isfinite(got[0]).all()) and float(got[0].abs().max()) > 0.0
    assert torch.equal(got[0], got[1]) and torch.equal(got[0], got[2])
