"""The sampler's elimination on many workgroups (buffers of 4,096 entries and
more) against the oracle: the same draws from the same conditionals, so the
configurations, their counts and their order are equal."""
import numpy as np
import pytest
import torch

from gen import init_params
from oracle import made, sampler

pytestmark = pytest.mark.gpu


# (n, n_up, n_dn, draws, buffer, std of the parameters): no elimination; a threshold
# found by one bin (small counts, many ties); by the listed counts of a bin; the
# smallest buffer; equal weights, where one bin holds more counts than the list;
# the conditionals in half and in whole tiles
@pytest.mark.parametrize("n,nu,nd,draws,umax,std", [
    (12, 3, 3, 10**9, 4500, 0.5), (13, -1, -1, 20000, 4500, 0.1), (13, -1, -1, 10**12, 4096, 0.5),
    (13, -1, -1, 10**12, 4500, 0.0), (14, -1, -1, 10**7, 4097, 0.3), (13, -1, -1, 3 * 10**5, 5000, 0.0),
    (14, -1, -1, 10**9, 8192, 0.3), (14, -1, -1, 10**9, 8193, 0.3)])
def test_shared_elimination_matches_oracle(n, nu, nd, draws, umax, std):
    import paper_2208_05637_amd as nqs
    nqs.load()
    print(f"sampler: n={n} sector=({nu},{nd}) draws={draws} buffer={umax} std={std}", flush=True)
    ctx = nqs.Context(0)
    H = nqs.Hamiltonian(n, [1], [0], [1.0]).upload(ctx)
    plan = nqs.Plan(ctx, H, 1, 64, nu, nd, "fp64", max_batch=16)
    params = init_params(n, 1, 64, seed=n, std=std)
    x, w = nqs.sample(plan, torch.from_numpy(params).cuda(), draws, seed=77, max_unique=umax)
    xr, cr = sampler.sample(made.Net(n=n, n_layers=1, width=64, n_up=nu, n_dn=nd), params, draws, seed=77, max_unique=umax)
    print(f"   {len(xr)} unique; GPU {len(x)}")
    assert np.array_equal(x.cpu().numpy().view(np.uint64), xr)
    assert np.array_equal(w.cpu().numpy(), cr.astype(np.float64))
