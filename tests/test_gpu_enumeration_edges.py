"""Connected configurations and their reduction at the edges of the kernels'
shares: diagonal terms in batches of 64, flips in ranges of a wave's width,
samples in workgroups of 16 and 64, reductions of one to eight slices.

The entries are whole numbers and single coefficients and the diagonal is a
sum in the terms' order, so both are equal to the reference's.  The reduction
is a compensated sum (one rounding) of products whose factors (exp, cos, sin,
the differences of log psi of size 4, three products) are within 16 eps
together.
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nqs():
    import paper_2208_05637_amd as m
    m.load()
    return m


def _words(v, n):
    return np.array(v, dtype=np.uint64) if n <= 64 else np.array([[a & (2**64 - 1), a >> 64] for a in v], dtype=np.uint64)


@pytest.mark.parametrize("n,terms,flips,B", [
    (12, 0, 1, 1), (12, 1, 63, 17), (24, 63, 64, 300), (24, 64, 65, 33), (40, 65, 1024, 600),
    (40, 130, 1025, 5), (64, 128, 2049, 3), (76, 100, 500, 64), (76, 64, 9000, 2)])
def test_entries_diagonal_and_sum(nqs, n, terms, flips, B):
    print(f"enumeration: n={n} diagonal terms={terms} flips={flips} samples={B}", flush=True)
    rng = np.random.default_rng(n + flips)
    word = lambda: sum(int(rng.integers(0, 2**32)) << (32 * k) for k in range(4)) & ((1 << n) - 1)
    fl = set()
    while len(fl) < flips:
        fl.add(sum(1 << int(q) for q in rng.choice(n, size=int(rng.integers(1, 5)), replace=False)))
    fl = sorted(fl)
    dz = set()
    while len(dz) < terms:
        dz.add(word())
    dz = sorted(dz)
    z = [word() & ~f for f in fl]
    coeff = rng.normal(size=terms + flips) * 10.0 ** rng.integers(-4, 4, size=terms + flips)
    ctx = nqs.Context(0)
    H = nqs.Hamiltonian(n, _words([0] * terms + fl, n), _words(dz + z, n), coeff, drop_tol=0.0,
                        conserves_spin=False).upload(ctx)
    plan = nqs.Plan(ctx, H, 1, 64, -1, -1, "fp64", max_batch=B)
    x = [word() for _ in range(B)]
    con = nqs.connected(plan, torch.from_numpy(_words(x, n).view(np.int64)).cuda())
    m = int(con["n_entries"].item())
    assert m == B * flips and nqs.device_status(plan) == 0
    sign = lambda a, b: -1.0 if bin(a & b).count("1") & 1 else 1.0
    diag = []
    for v in x:
        acc = 0.0
        for k in range(terms):
            acc += sign(v, dz[k]) * coeff[k]
        diag.append(acc)
    np.testing.assert_array_equal(con["diag"].cpu().numpy(), np.stack([diag, np.zeros(B)], 1))
    want_h = np.array([[sign(v, z[g]) * coeff[terms + g] for g in range(flips)] for v in x])
    np.testing.assert_array_equal(con["h"][:m, 0].cpu().numpy().reshape(B, flips), want_h)
    want_x = _words([v ^ f for v in x for f in fl], n)
    np.testing.assert_array_equal(con["x"][:m].cpu().numpy().view(np.uint64), want_x)
    lps = rng.uniform(-2, 2, size=(B, 2))
    lpe = rng.uniform(-2, 2, size=(m, 2))
    lpe[rng.random(m) < 0.1, 0] = -np.inf
    got = nqs.reduce_table(plan, torch.from_numpy(lps).cuda(), torch.from_numpy(lpe).cuda(), con["diag"],
                           con["sample"][:m], con["h"][:m], m).cpu().numpy()
    d = lpe.reshape(B, flips, 2) - lps[:, None, :]
    size = want_h * np.exp(d[..., 0])
    eps = 2.0**-52
    bar = 16 * eps * np.abs(size).sum(1) + 4 * eps * np.abs(diag)
    want = np.longdouble(np.stack([size * np.cos(d[..., 1]), size * np.sin(d[..., 1])], -1)).sum(1)
    want[:, 0] += diag
    assert (np.abs(got - want) <= bar[:, None]).all()


@pytest.mark.parametrize("n,B,every", [(12, 3, 1), (24, 70, 2), (24, 700, 1), (66, 40, 3)])
def test_groups_of_few_and_many_terms(nqs, n, B, every):
    """Flips within a spin, of one to eight terms or (every `every`-th) of nine
    to thirty, which a wave collects over its samples.  Coefficients are
    multiples of 2^-10, so that every sum is exact."""
    print(f"enumeration: n={n} samples={B}, long groups every {every}", flush=True)
    rng = np.random.default_rng(n + B)
    word = lambda: sum(int(rng.integers(0, 2**32)) << (32 * k) for k in range(4)) & ((1 << n) - 1)
    fl = sorted((1 << a) | (1 << b) for a in range(n) for b in range(a + 2, n, 2))
    xm, zm, cf, terms = [], [], [], []
    for k, f in enumerate(fl):
        count = int(rng.integers(9, 31)) if k % every == 0 else int(rng.integers(1, 9))
        zs = set()
        while len(zs) < count:
            zs.add(word() & ~f)
        c = rng.integers(1, 4096, size=count) * rng.choice([-1, 1], size=count) / 1024.0
        terms.append(list(zip(sorted(zs), c)))
        xm += [f] * count
        zm += sorted(zs)
        cf += list(c)
    ctx = nqs.Context(0)
    H = nqs.Hamiltonian(n, _words(xm, n), _words(zm, n), np.array(cf), drop_tol=0.0, conserves_spin=True).upload(ctx)
    nu, nd = n // 4, n // 6
    plan = nqs.Plan(ctx, H, 1, 64, nu, nd, "fp64", max_batch=B)
    x = [sum(1 << int(q) for q in 2 * rng.permutation(n // 2)[:nu]) +
         sum(1 << int(q) for q in 2 * rng.permutation(n // 2)[:nd] + 1) for _ in range(B)]
    con = nqs.connected(plan, torch.from_numpy(_words(x, n).view(np.int64)).cuda())
    m = int(con["n_entries"].item())
    assert nqs.device_status(plan) == 0
    wx, wh = [], []
    for v in x:
        for f, ts in zip(fl, terms):
            if bin(v & f).count("1") == 1:                                      # moves one particle
                wx.append(v ^ f)
                wh.append(sum(-c if bin(v & z).count("1") & 1 else c for z, c in ts))
    assert m == len(wx)
    np.testing.assert_array_equal(con["x"][:m].cpu().numpy().view(np.uint64), _words(wx, n))
    np.testing.assert_array_equal(con["h"][:m, 0].cpu().numpy(), np.array(wh))
