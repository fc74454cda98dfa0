"""Workspaces smaller than a call can use: the sizes that calls took before the
prefix states existed are still taken, nqs_*_workspace_least says how small one
may be, and the Python calls fall back to it where the device has no room."""
import ctypes as C

import numpy as np
import pytest
import torch

from gen import init_params

pytestmark = pytest.mark.gpu

TOO_SMALL = 4          # NQS_ERR_WORKSPACE_TOO_SMALL

N, LAYERS, WIDTH, FLIPS, BATCH = 24, 2, 256, 400, 3000
SIZE_BEFORE = 57993216


@pytest.fixture(scope="module")
def nqs():
    import paper_2208_05637_amd as m
    m.load()
    return m


@pytest.fixture(scope="module")
def case(nqs):
    """A plan whose connected configurations go down the prefix tree, its parameters and samples."""
    rng = np.random.default_rng(5)
    flips = [0] + sorted({int(v) for v in rng.integers(1, 1 << N, FLIPS)})
    z = [int(rng.integers(0, 1 << N)) & ~f for f in flips]
    ctx = nqs.Context(0)
    H = nqs.Hamiltonian(N, np.array(flips, dtype=np.uint64), np.array(z, dtype=np.uint64), rng.normal(size=len(flips)),
                        conserves_spin=False).upload(ctx)
    params = torch.from_numpy(init_params(N, LAYERS, WIDTH, seed=2)).cuda()
    x = torch.from_numpy(rng.integers(0, 1 << N, BATCH).astype(np.int64)).cuda()

    def plan():
        return nqs.Plan(ctx, H, LAYERS, WIDTH, -1, -1, "fp32", max_batch=BATCH, dedup=False)

    return plan, params, x


def _buffer(nb):
    raw = torch.empty(nb + 256, dtype=torch.uint8, device="cuda")
    return raw, C.c_void_p((raw.data_ptr() + 255) & ~255)


def _call(plan, params, x, nb):
    """nqs_local_energy with a workspace of nb bytes: (status, local energies)."""
    out = torch.full((x.shape[0], 2), float("nan"), dtype=torch.float64, device="cuda")
    raw, ws = _buffer(nb)
    st = plan.lib.nqs_local_energy(plan.handle, C.c_void_p(params.data_ptr()), C.c_void_p(x.data_ptr()), x.shape[0],
                                   C.c_void_p(out.data_ptr()), ws, nb)
    torch.cuda.synchronize()
    return st, out


def test_least_workspace_is_taken_and_no_less(nqs, case):
    make, params, x = case
    plan = make()
    full, least = plan.workspace_size(BATCH), plan.workspace_size(BATCH, least=True)
    assert least < full
    want = nqs.local_energy(plan, params, x)
    for nb in (full, least + (full - least) // 2, least + 1, least):
        st, got = _call(plan, params, x, nb)
        assert st == 0
        torch.testing.assert_close(got, want, rtol=1e-12, atol=1e-12)
    assert _call(plan, params, x, least - 1)[0] == TOO_SMALL


def test_size_from_before_the_prefix_states(nqs, case):
    """What this plan's workspace measured when every forward ran row by row."""
    make, params, x = case
    assert make().workspace_size(BATCH, least=True) <= SIZE_BEFORE
    assert _call(make(), params, x, SIZE_BEFORE)[0] == 0


def test_profile_of_a_smaller_batch(nqs, case):
    """The flops of profiled launches, whose place behind the workspace depends on the batch."""
    make, params, x = case
    plan = make()
    plan.workspace()
    done = []
    for B in (BATCH, BATCH - 777, BATCH):
        plan.profile(True)
        nqs.local_energy(plan, params, x[:B])
        r = plan.profile_read()
        assert r["forward_launches"] == 2 and r["forward_rows"] == B * (plan.entries_per_sample + 1)
        done.append(r["forward_flops_executed"] / r["forward_rows"])
    assert done[0] == done[2] and 0.5 < done[1] / done[0] < 2.0
    plan.workspace(least=True)
    plan.profile(True)
    nqs.local_energy(plan, params, x)
    assert plan.profile_read()["forward_flops_executed"] / (BATCH * (plan.entries_per_sample + 1)) > 1.2 * done[0]


@pytest.mark.parametrize("share", [0.0, 0.3, 0.6, 1.0])
def test_multi_with_part_of_the_states(nqs, case, share):
    make, params, x = case
    items, single = [], []
    for B in (BATCH, BATCH // 2):
        p = make()
        single.append([t.clone() for t in nqs.energy_grad(p, params, x[:B].contiguous())])
        items.append(dict(plan=p, params=params, samples=x[:B].contiguous(), weights=None,
                          eloc=torch.empty((B, 2), dtype=torch.float64, device="cuda"),
                          energy=torch.empty(3, dtype=torch.float64, device="cuda"),
                          grad=torch.empty(p.n_params, dtype=torch.float64, device="cuda")))
    lib = nqs.load()
    from paper_2208_05637_amd.api import _instances
    full, least = C.c_size_t(), C.c_size_t()
    assert lib.nqs_multi_workspace_size(2, _instances(items), C.byref(full)) == 0
    assert lib.nqs_multi_workspace_least(2, _instances(items), C.byref(least)) == 0
    assert least.value < full.value and least.value == sum(
        it["plan"].workspace_size(it["samples"].shape[0], least=True) for it in items)
    nb = least.value + int(share * (full.value - least.value))
    raw, ws = _buffer(nb)
    nqs.energy_grad_multi(items, (raw, ws, nb))
    assert nqs.multi_device_status(items, (raw, ws, nb)) == 0
    for it, (energy, grad, eloc) in zip(items, single):
        torch.testing.assert_close(it["eloc"], eloc, rtol=1e-12, atol=1e-12)
        torch.testing.assert_close(it["grad"], grad, rtol=1e-5, atol=1e-9)
    raw, ws = _buffer(least.value)
    assert lib.nqs_energy_grad_multi(2, _instances(items), ws, least.value - 1) == TOO_SMALL


def _no_room(monkeypatch, most):
    real = torch.empty

    def empty(*a, **k):
        if k.get("dtype") is torch.uint8 and a[0] > most:
            raise torch.OutOfMemoryError("no room")
        return real(*a, **k)

    monkeypatch.setattr(torch, "empty", empty)


def test_python_falls_back_where_there_is_no_room(nqs, case, monkeypatch):
    make, params, x = case
    want = nqs.local_energy(make(), params, x)
    plan = make()
    least = plan.workspace_size(BATCH, least=True)
    _no_room(monkeypatch, least + 256)
    got = nqs.local_energy(plan, params, x)
    torch.testing.assert_close(got, want, rtol=1e-12, atol=1e-12)
    assert plan.workspace()[1] == least
    monkeypatch.undo()
    assert plan.workspace()[1] == least                        # the plan keeps to it ...
    assert plan.workspace(least=False)[1] > least              # ... until it is told otherwise
    _no_room(monkeypatch, least // 2)
    with pytest.raises(torch.OutOfMemoryError):
        nqs.local_energy(make(), params, x)


def test_sampler_falls_back_where_there_is_no_room(nqs, case, monkeypatch):
    make, params, _ = case
    plan = make()
    want = nqs.sample(plan, params, 10**9, 3, 500)
    size, least = C.c_size_t(), C.c_size_t()
    assert plan.lib.nqs_sample_workspace_size(plan.handle, 500, C.byref(size)) == 0
    assert plan.lib.nqs_sample_workspace_least(plan.handle, 500, C.byref(least)) == 0
    assert least.value < size.value
    _no_room(monkeypatch, least.value + 256)
    got = nqs.sample(plan, params, 10**9, 3, 500)
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
