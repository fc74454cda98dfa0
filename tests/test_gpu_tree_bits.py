"""The two forwards of the connected configurations give equal bits: local
energies down the prefix tree (a full workspace, and part of its states) and row
by row (the least workspace) are the same doubles, for every kind, workgroup
shape, word count, with and without hash tables, chunk by chunk and in one.  That
the full workspace takes the tree and the least does not is read off the matrix
operations that the profile counts."""
import ctypes as C
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


def _words(ints, n):
    if n <= 64:
        return np.array(ints, dtype=np.uint64)
    return np.array([[v & (2**64 - 1), v >> 64] for v in ints], dtype=np.uint64)


def _problem(nqs, n, G, sector, B, seed):
    """A Hamiltonian of G flips of up to four qubits and B samples (some of them equal)."""
    rng = np.random.default_rng(seed)
    flips = set()
    while len(flips) < min(G, sum(math.comb(n, k) for k in range(1, 5)) // 2):
        flips.add(sum(1 << int(q) for q in rng.choice(n, size=int(rng.integers(1, 5)), replace=False)))
    flips = [0] + sorted(flips)
    z = [int(rng.integers(0, 2**62)) & ((1 << n) - 1) & ~f for f in flips]
    ctx = nqs.Context(0)
    H = nqs.Hamiltonian(n, _words(flips, n), _words(z, n), rng.normal(size=len(flips)), conserves_spin=False).upload(ctx)
    nu, nd = ((n + 1) // 4, n // 4) if sector else (-1, -1)
    xs = []
    for _ in range(min(B, 4000)):
        if sector:
            v = sum(1 << int(q) for q in 2 * rng.permutation((n + 1) // 2)[:nu])
            v |= sum(1 << int(q) for q in 2 * rng.permutation(n // 2)[:nd] + 1)
        else:
            v = sum(1 << int(q) for q in np.nonzero(rng.random(n) < 0.5)[0])
        xs.append(v)
    xs = sorted(xs)
    w = _words([xs[i * len(xs) // B] for i in range(B)], n)
    return ctx, H, nu, nd, torch.from_numpy(w.view(np.int64)).cuda()


def _eloc(plan, params, x, nb):
    """Local energies with a workspace of nb bytes, and the MFMA flops issued for them."""
    out = torch.empty((x.shape[0], 2), dtype=torch.float64, device="cuda")
    raw = torch.empty(nb + 256, dtype=torch.uint8, device="cuda")
    ws = C.c_void_p((raw.data_ptr() + 255) & ~255)
    plan.profile(True)
    assert plan.lib.nqs_local_energy(plan.handle, C.c_void_p(params.data_ptr()), C.c_void_p(x.data_ptr()), x.shape[0],
                                     C.c_void_p(out.data_ptr()), ws, nb) == 0
    from paper_2208_05637_amd import _lib
    prof = _lib.Profile()
    assert plan.lib.nqs_plan_profile_read(plan.handle, ws, C.byref(prof)) == 0
    plan.profile(False)
    return out, prof.forward_flops_executed


# (n, precision, width, layers, flips, phase_mode, sector, samples)
CASES = [
    (24, "fp64", 128, 2, 300, 0, True, 4000),
    (28, "fp64", 256, 3, 300, 1, False, 800),
    (76, "fp64", 256, 2, 300, 0, True, 1500),
    (33, "fp64", 512, 2, 400, 0, False, 400),
    (60, "fp64", 1024, 2, 300, 0, True, 300),
    (40, "fp32", 128, 2, 300, 0, True, 6000),
    (33, "fp32", 256, 2, 400, 0, False, 2000),
    (28, "fp32", 256, 3, 200, 1, True, 3000),
    (64, "fp32", 512, 3, 300, 0, True, 1000),
    (65, "fp32", 1024, 2, 300, 0, False, 800),
    (60, "bf16", 256, 3, 400, 0, False, 6000),
    (41, "bf16", 512, 3, 500, 0, True, 2000),
    (100, "bf16", 1024, 4, 400, 0, True, 2000),
    (36, "bf16x3", 256, 2, 400, 1, True, 4000),
    (64, "bf16x3", 512, 3, 400, 0, False, 1000),
    (65, "bf16x3", 1024, 2, 400, 0, True, 800),
    (60, "bf16w", 256, 3, 700, 0, False, 4000),
    (40, "bf16w", 512, 3, 700, 0, True, 1000),
    (128, "bf16w", 512, 2, 600, 1, False, 1000),
    (60, "bf16w", 1024, 4, 700, 0, True, 900),
    (76, "bf16w", 1024, 2, 600, 0, False, 1500),
]


@pytest.mark.parametrize("n,prec,h,L,G,phase,sector,B", CASES)
def test_same_bits(nqs, n, prec, h, L, G, phase, sector, B):
    ctx, H, nu, nd, x = _problem(nqs, n, G, sector, B, 17 * n + h)
    params = torch.from_numpy(init_params(n, L, h, seed=3, phase_mode=phase)).cuda()
    plan = nqs.Plan(ctx, H, L, h, nu, nd, prec, max_batch=B, dedup=False, phase_mode=phase)
    full, least = plan.workspace_size(B), plan.workspace_size(B, least=True)
    shapes = {}
    base = plan.kernel_info()
    for waves in (8, 16):
        for rows in (base["rows_per_block"], base["rows_per_block"] // 2):
            try:
                plan.configure(waves_per_block=waves, rows_per_block=rows)
            except nqs._lib.NQSError:
                continue
            shapes[waves, rows] = None
    assert (base["waves_per_block"], base["rows_per_block"]) in shapes
    for waves, rows in shapes:
        print(f"n={n} {prec} h={h} L={L} phase={phase} sector={sector} B={B}: {waves} waves, {rows} rows", flush=True)
        plan.configure(waves_per_block=waves, rows_per_block=rows)
        rowwise, f0 = _eloc(plan, params, x, least)
        tree, f1 = _eloc(plan, params, x, full)
        part, f2 = _eloc(plan, params, x, least + int(0.85 * (full - least)))
        assert f1 != f0 and f2 != f0                           # other matrix operations: the tree ran
        assert bool(torch.isfinite(rowwise).all())
        assert torch.equal(tree, rowwise) and torch.equal(part, rowwise)


@pytest.mark.parametrize("n,prec,h,L,phase,sector", [
    (40, "bf16w", 512, 3, 0, True), (33, "fp32", 256, 2, 1, False), (26, "fp64", 256, 2, 0, True),
    (70, "bf16w", 1024, 2, 0, False), (63, "bf16", 512, 3, 0, False)])
@pytest.mark.parametrize("distinct", [1, 3, 41])
def test_same_bits_with_few_rows(nqs, n, prec, h, L, phase, sector, distinct):
    """Hash tables and many equal samples: the call's bound takes the tree, which then has one node, a few, or
    tiles that are nearly empty; also in two chunks, whose second has the look-back's rows only, and in a long and
    a short chunk, which may take different forwards."""
    B, G = 3000, 400
    ctx, H, nu, nd, x = _problem(nqs, n, G, sector, distinct, n + distinct)
    x = x.repeat_interleave(B // distinct, dim=0).contiguous()
    B = x.shape[0]
    params = torch.from_numpy(init_params(n, L, h, seed=4, phase_mode=phase)).cuda()
    ref = nqs.Plan(ctx, H, L, h, nu, nd, prec, max_batch=B, dedup=False, phase_mode=phase)
    want, _ = _eloc(ref, params, x, ref.workspace_size(B, least=True))
    for chunk in (B, (B + 1) // 2, B - 5):
        plan = nqs.Plan(ctx, H, L, h, nu, nd, prec, max_batch=B, dedup=True, phase_mode=phase, chunk_samples=chunk)
        got, f1 = _eloc(plan, params, x, plan.workspace_size(B))
        low, f0 = _eloc(plan, params, x, plan.workspace_size(B, least=True))
        assert f1 != f0
        print(f"n={n} {prec} h={h} distinct={distinct} chunk={chunk} of {B}", flush=True)
        assert torch.equal(got, want) and torch.equal(low, want)


def test_same_bits_allocation_free(nqs):
    """The 256 MB call has states for part of the workgroups, or none, where the workspace call has all."""
    ctx, H, nu, nd, x = _problem(nqs, 40, 300, True, 900, 9)
    params = torch.from_numpy(init_params(40, 3, 512, seed=3)).cuda()
    plan = nqs.Plan(ctx, H, 3, 512, nu, nd, "bf16w", max_batch=900, dedup=False)
    assert plan.workspace_size(900) > nqs._lib.NQS_NOALLOC_SCRATCH_BYTES > plan.workspace_size(900, least=True)
    e0, g0, l0 = nqs.energy_grad(plan, params, x)
    e1, g1, l1, flags = nqs.energy_grad_noalloc(plan, params, x)
    assert int(flags.item()) == 0
    assert torch.equal(l0, l1) and torch.equal(e0, e1)
