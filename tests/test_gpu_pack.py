"""Packed weights where their order is unusual: fewer units than degrees (a unit
per class, and classes without one), two qubits, one and two words, uneven
classes, both phase networks, a sampling order of its own; log psi against the
oracle within the bars of the same arithmetic at 12 qubits."""
import numpy as np
import pytest
import torch

from gen import init_params
from oracle import made

pytestmark = pytest.mark.gpu
TOL = {"fp64": 1e-12, "fp32": 2e-5, "bf16x3": 5e-4, "bf16w": 5e-4}


@pytest.mark.parametrize("n,prec,h,L,phase", [
    (2, "fp64", 64, 2, 0), (3, "fp32", 128, 1, 0), (64, "fp64", 64, 2, 0), (65, "fp64", 64, 3, 0),
    (66, "fp64", 64, 2, 1), (128, "fp64", 64, 2, 0), (100, "fp64", 128, 2, 1), (100, "fp32", 256, 2, 0),
    (33, "bf16x3", 256, 3, 1), (127, "bf16w", 512, 2, 0), (44, "bf16x3", 512, 3, 0)])
@pytest.mark.parametrize("shuffled", [False, True])
def test_log_psi_of_packed_weights(n, prec, h, L, phase, shuffled):
    import paper_2208_05637_amd as nqs
    nqs.load()
    print(f"packing: n={n} {prec} h={h} L={L} phase={phase} shuffled={shuffled}", flush=True)
    rng = np.random.default_rng(n + h)
    order = rng.permutation(n) if shuffled else None
    one = np.array([1], dtype=np.uint64) if n <= 64 else np.array([[1, 0]], dtype=np.uint64)
    H = nqs.Hamiltonian(n, one, one * np.uint64(0), np.ones(1), conserves_spin=False).upload(ctx := nqs.Context(0))
    plan = nqs.Plan(ctx, H, L, h, -1, -1, prec, max_batch=4, order=order, phase_mode=phase)
    params = init_params(n, L, h, seed=5, std=0.1, dtype="bf16" if prec == "bf16w" else "fp32", phase_mode=phase)
    xs = rng.integers(0, 2**63, size=(70, (n + 63) // 64)).astype(np.uint64) * 2 + 1
    xs[:, -1] &= np.uint64((1 << ((n - 1) % 64 + 1)) - 1)
    xs = xs[:, 0] if n <= 64 else xs
    net = made.Net(n=n, n_layers=L, width=h, order=order, phase_mode=phase)
    la, ph, _ = made.forward(net, params, xs)
    out = nqs.log_psi(plan, torch.from_numpy(params).cuda(), torch.from_numpy(xs.view(np.int64)).cuda()).cpu().numpy()
    assert np.abs(out[:, 0] - la).max() <= TOL[prec] and np.abs(out[:, 1] - ph).max() <= TOL[prec]
