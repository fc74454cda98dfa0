"""Which forward the connected configurations of a call take: the prefix tree only
where its handful of tiles per workgroup is faster than the rows one by one.  Read
off the matrix operations that the profile counts, against the same call with the
least workspace, which goes row by row.  Both forwards were timed at these points."""
import ctypes as C

import numpy as np
import pytest
import torch

from gen import init_params
from gen.inputs import hamiltonian, sector_samples, unique_with_counts

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nqs():
    import paper_2208_05637_amd as m
    m.load()
    return m


# (orbitals, layers, width, precision, phase_mode, samples, down the tree): us row by row | down the tree (no case
# has so many entries that its sector is indexed)
CASES = [
    (9, 4, 1024, "bf16w", 0, 30, False),        # 227 | 463 (20,000 rows at 16 qubits)
    (10, 4, 1024, "bf16w", 0, 24, False),
    (10, 4, 1024, "bf16w", 1, 24, False),       # (the phase network's cost does not count)
    (12, 4, 1024, "bf16", 0, 40, False),        # 383 | 523
    (12, 1, 64, "fp64", 0, 200, False),         # 231 | 283
    (12, 2, 256, "bf16w", 0, 40, False),        # 87 | 102
    (12, 1, 128, "fp32", 0, 200, False),        # 180 | 207
    (12, 3, 512, "fp32", 0, 200, True),         # 2,248 | 1,183
    (12, 4, 1024, "bf16w", 0, 200, True),       # 2,584 | 1,845
    (12, 3, 256, "fp64", 0, 80, True),          # 639 | 442
    (12, 3, 512, "bf16w", 1, 100, True),        # 327 | 216
    (12, 2, 1024, "bf16x3", 0, 100, True),      # 850 | 551
]


def _flops(plan, params, x, nb):
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


@pytest.mark.parametrize("orbitals,layers,width,precision,phase,samples,tree", CASES)
def test_route(nqs, orbitals, layers, width, precision, phase, samples, tree):
    n, ne = 2 * orbitals, orbitals // 2
    ctx = nqs.Context(0)
    H = nqs.Hamiltonian.from_terms(hamiltonian(orbitals, 0)).upload(ctx)
    params = torch.from_numpy(init_params(n, layers, width, seed=1, phase_mode=phase)).cuda()
    x, _ = unique_with_counts(sector_samples(n, ne, ne, samples, seed=2))
    x = torch.from_numpy(np.resize(x, samples).view(np.int64)).cuda()
    plan = nqs.Plan(ctx, H, layers, width, ne, ne, precision, max_batch=100 * samples, dedup=False, phase_mode=phase,
                    chunk_samples=samples)
    # (a plan of a larger chunk keeps states for the tree, whatever this call needs)
    big = nqs.Plan(ctx, H, layers, width, ne, ne, precision, max_batch=100 * samples, dedup=False, phase_mode=phase)
    for p in (plan, big):
        e0, f0 = _flops(p, params, x, p.workspace_size(samples, least=True))
        e1, f1 = _flops(p, params, x, p.workspace_size(samples))
        print(f"{n} qubits, L={layers}, {width} {precision}, {samples} samples: tree {f1 != f0}", flush=True)
        assert (f1 != f0) == tree
        assert torch.equal(e0, e1)


@pytest.mark.parametrize("orbitals,cutoff,precision,chunk", [(12, 0.0, "bf16x3", 128), (38, 0.02, "bf16w", 32)])
def test_tuned_plans_of_the_tuner_tests(nqs, orbitals, cutoff, precision, chunk):
    """Two plans as the autotuner's tests use them (24 qubits; 76, of fewer strings there): their chunks go down the
    tree, so the candidates' shapes differ by the head's k slices and no more."""
    n, ne = 2 * orbitals, orbitals // 2
    ctx = nqs.Context(0)
    H = nqs.Hamiltonian.from_terms(hamiltonian(orbitals, 0, cutoff=cutoff)).upload(ctx)
    params = torch.from_numpy(init_params(n, 2, 512, seed=5)).cuda()
    x, _ = unique_with_counts(sector_samples(n, ne, ne, 2 * chunk, seed=4))
    x = torch.from_numpy(np.resize(x, (2 * chunk,) + x.shape[1:]).view(np.int64)).cuda()
    plan = nqs.Plan(ctx, H, 2, 512, ne, ne, precision, max_batch=2 * chunk, dedup="auto", chunk_samples=chunk)
    e0, f0 = _flops(plan, params, x, plan.workspace_size(2 * chunk, least=True))
    e1, f1 = _flops(plan, params, x, plan.workspace_size(2 * chunk))
    assert f1 != f0 and torch.equal(e0, e1)
