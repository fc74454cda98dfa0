"""The prefix-shared forward of the connected configurations against the
row-by-row forward: nqs_local_energy (which walks the prefix tree) and the same
local energies put together from nqs_connected, nqs_log_psi on every entry (row
by row) and nqs_reduce_table.

The logits and phases of the two forwards are equal, so log|psi| differs only
by the order of a sum of at most n log-sigmoids in FP64: by (n - 1) eps times
the sum of their magnitudes, |2 log|psi||, on either side, and E_loc by that
much of sum_e |h_e| |psi(x'_e) / psi(x)| (twice: the sample's amplitude too).
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


def _words(ints, n):
    if n <= 64:
        return np.array(ints, dtype=np.uint64)
    return np.array([[v & (2**64 - 1), v >> 64] for v in ints], dtype=np.uint64)


def _flips(n, count, rng):
    """Distinct non-empty flips of up to four qubits."""
    out = set()
    while len(out) < count:
        out.add(sum(1 << int(q) for q in rng.choice(n, size=min(n, int(rng.integers(1, 5))), replace=False)))
    return sorted(out)


# (n, precision, width, layers, flips, phase_mode, sector, batches): tile and
# block edges of each kind, one node and many, one and two words, L = 1 (no
# hidden layer), both sides of the rule for the cuts (width 512 | 1024).  The
# plan's chunk is large enough for the tree (about 100 us of the row-by-row
# forward); the batches go from one sample to segments long enough for a
# level's two tiles of states to be reused many times.
CASES = [
    (5, "fp64", 64, 1, 15, 0, False, (1, 3, 32)),
    (12, "fp64", 128, 2, 100, 0, True, (1, 200)),
    (33, "fp64", 256, 3, 500, 0, False, (7, 300)),
    (76, "fp64", 64, 2, 300, 0, True, (1, 700)),
    (60, "fp64", 1024, 2, 300, 0, False, (4,)),
    (24, "fp32", 128, 2, 300, 0, True, (37, 900)),
    (33, "fp32", 512, 1, 333, 0, False, (30,)),
    (64, "fp32", 1024, 2, 500, 0, False, (5,)),
    (28, "fp32", 256, 3, 200, 1, True, (1, 400)),
    (60, "bf16", 256, 2, 400, 0, False, (33,)),
    (100, "bf16", 1024, 2, 400, 0, True, (5,)),
    (64, "bf16x3", 512, 3, 400, 1, False, (2, 60)),
    (24, "bf16x3", 1024, 2, 300, 0, True, (9,)),
    (60, "bf16w", 1024, 4, 700, 0, True, (1, 60)),
    (65, "bf16w", 512, 2, 500, 0, False, (20,)),
    (128, "bf16w", 1024, 2, 600, 1, False, (8,)),
    (63, "bf16w", 256, 1, 64, 0, False, (17, 3000)),
    (40, "bf16w", 256, 2, 7000, 0, False, (700,)),
]


@pytest.mark.parametrize("n,prec,h,L,G,phase,sector,batches", CASES)
@pytest.mark.parametrize("dedup", [False, True])
def test_tree_equals_row_by_row(nqs, n, prec, h, L, G, phase, sector, batches, dedup):
    rng = np.random.default_rng(n * 1000 + h)
    G = min(G, sum(math.comb(n, k) for k in range(1, 5)) // 2)
    flips = [0] + _flips(n, G, rng)
    z = [int(rng.integers(0, 2**62)) & ((1 << n) - 1) & ~f for f in flips]      # no Y: real coefficients
    ctx = nqs.Context(0)
    H = nqs.Hamiltonian(n, _words(flips, n), _words(z, n), rng.normal(size=len(flips)), conserves_spin=False).upload(ctx)
    nu, nd = ((n + 1) // 4, n // 4) if sector else (-1, -1)
    params = torch.from_numpy(init_params(n, L, h, seed=3, phase_mode=phase)).cuda()
    plan = nqs.Plan(ctx, H, L, h, nu, nd, prec, max_batch=max(*batches, 600_000 // G), dedup=dedup, phase_mode=phase)
    ref = nqs.Plan(ctx, H, L, h, nu, nd, prec, max_batch=max(batches), phase_mode=phase)
    for B in batches:
        print(f"tree forward: n={n} {prec} h={h} L={L} B={B} flips={G} phase={phase} dedup={dedup}", flush=True)
        xs = set()
        while len(xs) < B:
            if sector:
                v = sum(1 << int(q) for q in 2 * rng.permutation((n + 1) // 2)[:nu])
                v |= sum(1 << int(q) for q in 2 * rng.permutation(n // 2)[:nd] + 1)
            else:
                v = sum(1 << int(q) for q in np.nonzero(rng.random(n) < 0.5)[0])
            xs.add(v)
        x = torch.from_numpy(_words(sorted(xs), n).view(np.int64)).cuda()
        got = nqs.local_energy(plan, params, x)
        assert nqs.device_status(plan) == 0
        con = nqs.connected(ref, x)
        m = int(con["n_entries"].item())
        lps = nqs.log_psi(ref, params, x)
        lpe = nqs.log_psi(ref, params, con["x"][:m].contiguous())
        want = nqs.reduce_table(ref, lps, lpe, con["diag"], con["sample"][:m], con["h"][:m], m)
        es = con["sample"][:m].long()
        size = con["h"][:m, 0].abs() * torch.exp(lpe[:, 0] - lps[es, 0])
        worst = torch.where(torch.isfinite(lpe[:, 0]), lpe[:, 0].abs(), torch.zeros_like(size)) + lps[es, 0].abs()
        eps = 2.0**-52
        bar = torch.zeros(B, dtype=torch.float64, device=x.device)
        bar.index_add_(0, es, size * (16 * eps + 2 * n * eps * worst))
        bar += 8 * eps * con["diag"][:, 0].abs()
        err = (got - want).abs().amax(dim=1)
        print(f"   {m} entries, largest error {float((err / bar).max()):.2e} of the bar", flush=True)
        assert bool(torch.isfinite(got).all()) and bool((err <= bar).all())
