"""The gradient's sums over samples, cut into blocks of 256 (FP32) or 64 (FP64)
samples: with room for the blocks' sums they run side by side, in batches where
only some fit, and without room one after the other.  All give the same bits,
and the FP64 oracle's gradient.

The Hamiltonian has no flips, so a plan without dedup has a few kilobytes of
local-energy buffers (no room) and one with dedup two small hash tables (room
for some blocks) for the same local energies.  Bars: those of the parity tests,
1e-9 relative for FP64 and 2e-5 for FP32 arithmetic (chains of at most 256
FP32 products, 256 * 2^-24 = 1.5e-5 if every rounding had one sign).
"""
import numpy as np
import pytest
import torch

from gen import init_params
from oracle import made, vmc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B", [1, 63, 64, 65, 255, 256, 257, 600])
@pytest.mark.parametrize("prec,h,L,n,phase", [("fp64", 64, 2, 11, 0), ("fp32", 128, 2, 13, 0), ("fp32", 128, 1, 13, 1)])
def test_blocks_of_samples(prec, h, L, n, phase, B):
    import paper_2208_05637_amd as nqs
    print(f"blocks: {prec} h={h} L={L} n={n} B={B}", flush=True)
    rng = np.random.default_rng(B)
    ctx = nqs.Context(0)
    z = np.arange(1, n + 1, dtype=np.uint64)
    H = nqs.Hamiltonian(n, np.zeros(n, dtype=np.uint64), z, rng.normal(size=n)).upload(ctx)
    xs = np.sort(rng.permutation(1 << n)[:B]).astype(np.uint64)
    w = rng.random(B) + 0.5
    params = init_params(n, L, h, seed=4, phase_mode=phase)
    p = torch.from_numpy(params).cuda()
    out = []
    for dedup in (False, True):
        plan = nqs.Plan(ctx, H, L, h, -1, -1, prec, max_batch=B, dedup=dedup, phase_mode=phase)
        e, g, el = nqs.energy_grad(plan, p, xs, w)
        out.append((e.cpu().numpy(), g.cpu().numpy(), el.cpu().numpy()))
    assert all(np.array_equal(a, b) for a, b in zip(*out))
    e, g, el = out[0]
    net = made.Net(n=n, n_layers=L, width=h, phase_mode=phase)
    ref = vmc.gradient(net, params, xs, w, el[:, 0] + 1j * el[:, 1], e[0])
    assert np.linalg.norm(g - ref) <= (1e-9 if prec == "fp64" else 2e-5) * np.linalg.norm(ref) + 1e-14
