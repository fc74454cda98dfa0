"""The sampler's walk in whole tiles (buffers of more than 64 entries per CU), whose
entries take their ancestors' states, against the whole network at every position
(the least workspace): the same configurations and counts."""
import ctypes as C

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


def _draw(plan, params, buf, nb):
    W = plan.words
    x = torch.zeros((buf, W), dtype=torch.int64, device="cuda")
    w = torch.zeros(buf, dtype=torch.float64, device="cuda")
    nu = torch.zeros(1, dtype=torch.int64, device="cuda")
    raw = torch.empty(nb + 256, dtype=torch.uint8, device="cuda")
    ws = C.c_void_p((raw.data_ptr() + 255) & ~255)
    assert plan.lib.nqs_sample(plan.handle, C.c_void_p(params.data_ptr()), 10**12, 11, buf, C.c_void_p(x.data_ptr()),
                               C.c_void_p(w.data_ptr()), C.c_void_p(nu.data_ptr()), ws, nb) == 0
    return int(nu.item()), x, w


@pytest.mark.parametrize("n,prec,h,L,sector,buf", [
    (60, "bf16w", 512, 3, True, 16385),
    (100, "bf16w", 1024, 2, True, 20000),
    (40, "bf16w", 256, 2, False, 33333),
    (40, "fp32", 256, 2, True, 20000),
    (70, "fp32", 512, 2, False, 17000),
    (44, "bf16x3", 512, 2, True, 20011),
    (60, "bf16", 512, 3, False, 16400),
    (36, "fp64", 256, 2, True, 9001),
])
def test_whole_tiles_draw_the_same(nqs, n, prec, h, L, sector, buf):
    ctx = nqs.Context(0)
    W = (n + 63) // 64
    f = np.zeros((2, W), dtype=np.uint64)
    f[1, 0] = 5
    shape = (lambda a: a if W == 2 else a[:, 0].copy())
    H = nqs.Hamiltonian(n, shape(f), shape(np.zeros_like(f)), np.ones(2), conserves_spin=False).upload(ctx)
    nu, nd = ((n + 1) // 4, n // 4) if sector else (-1, -1)
    plan = nqs.Plan(ctx, H, L, h, nu, nd, prec, max_batch=1, dedup=False)
    params = torch.from_numpy(init_params(n, L, h, seed=6)).cuda()
    size, least = C.c_size_t(), C.c_size_t()
    assert plan.lib.nqs_sample_workspace_size(plan.handle, buf, C.byref(size)) == 0
    assert plan.lib.nqs_sample_workspace_least(plan.handle, buf, C.byref(least)) == 0
    assert least.value < size.value                            # the walk has states to keep
    u0, x0, w0 = _draw(plan, params, buf, least.value)
    u1, x1, w1 = _draw(plan, params, buf, size.value)
    print(f"n={n} {prec} h={h} buffer {buf}: {u0} entries", flush=True)
    assert u0 == u1 and u0 > buf // 2
    assert torch.equal(x0[:u0], x1[:u0]) and torch.equal(w0[:u0], w1[:u0])
