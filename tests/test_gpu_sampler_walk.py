"""The sampler's two ways through a buffer, draw for draw: entries carried from
level to level of the prefix tree, and (with a workspace that has no room for
their states) the whole network row by row at every position.  The conditional
logits are equal, so the buffers are, with and without elimination (ties at the
threshold among them: few draws in a large buffer).
"""
import ctypes as C

import numpy as np
import pytest
import torch

from gen import init_params

pytestmark = pytest.mark.gpu

# (n, precision, width, layers, electrons, draws, buffer): level and tile edges
# of each kind, one and two words, buffers below, at and above a tile and above
# one pass of the fold's workgroup, draws from a handful to 10^12
CASES = [
    (6, "fp64", 64, 1, (2, 1), 1000, 3),
    (13, "fp64", 256, 2, (-1, -1), 200, 64),
    (20, "fp64", 128, 1, (5, 5), 10**6, 33),
    (24, "fp32", 128, 2, (6, 6), 10**12, 1000),
    (31, "fp32", 512, 3, (-1, -1), 5000, 4096),
    (40, "bf16", 256, 2, (10, 10), 10**9, 65),
    (64, "bf16x3", 512, 2, (20, 11), 10**7, 129),
    (60, "bf16w", 1024, 3, (15, 15), 10**12, 2500),
    (76, "bf16w", 512, 2, (19, 19), 10**12, 700),
    (128, "bf16w", 1024, 2, (-1, -1), 10**5, 300),
]


@pytest.mark.parametrize("n,prec,h,L,ne,draws,buf", CASES)
def test_walk_equals_row_by_row(n, prec, h, L, ne, draws, buf):
    import paper_2208_05637_amd as nqs
    print(f"sampler walk: n={n} {prec} h={h} L={L} draws={draws} buffer={buf}", flush=True)
    ctx = nqs.Context(0)
    one = (np.uint64(0),) if n <= 64 else (np.uint64(0), np.uint64(0))
    x = np.array(one, dtype=np.uint64).reshape(1) if n <= 64 else np.array([one], dtype=np.uint64)
    z = x.copy()
    z.reshape(-1)[0] = 1
    H = nqs.Hamiltonian(n, x, z, np.ones(1)).upload(ctx)
    p = torch.from_numpy(init_params(n, L, h, seed=5, std=0.05)).cuda()
    plan = nqs.Plan(ctx, H, L, h, *ne, prec, max_batch=1)
    xs, w = nqs.sample(plan, p, draws, seed=9, max_unique=buf)
    need = C.c_size_t()
    assert plan.lib.nqs_sample_workspace_size(plan.handle, buf, C.byref(need)) == 0
    raw = torch.empty(need.value + 256, dtype=torch.uint8, device="cuda")
    ws = C.c_void_p((raw.data_ptr() + 255) & ~255)
    x2 = torch.zeros(buf if n <= 64 else (buf, 2), dtype=torch.int64, device="cuda")
    w2 = torch.zeros(buf, dtype=torch.float64, device="cuda")
    nu = torch.zeros(1, dtype=torch.int64, device="cuda")
    ptr = lambda t: C.c_void_p(t.data_ptr())
    assert plan.lib.nqs_sample(plan.handle, ptr(p), draws, 9, buf, ptr(x2), ptr(w2), ptr(nu), ws, need.value - 256) == 0
    U = int(nu.item())
    print(f"   {U} configurations, {float(w.sum()):.6g} draws", flush=True)
    assert U == len(w) and torch.equal(xs, x2[:U]) and torch.equal(w, w2[:U])
