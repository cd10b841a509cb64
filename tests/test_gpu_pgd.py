"""GPU nominal-point refinement (leb_pgd_nominal) against the oracle's
(oracle/pgd.py) on the planar quadrotor and chains, both readings of the
covered set, and against random nominal points at an equal GPU time budget
(the comparison of the paper's Table II)."""
import time

import numpy as np
import pytest

import workloads as W
from parity import check_bounds

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    import paper_2607_01203_amd as leb
    leb.lib()
    return torch.device("cuda:0")


def _t(a, dev):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).to(dev)


def _case(name):
    if name == "planar_quad":
        return W.planar_quad_cfg(N=16)
    if name == "chain4":
        return W.chain_batch(31, 2, 7, 4)
    return W.chain_batch(32, 1, 5, 28)


def _offcentre(b, seed, frac=0.5):
    rng = np.random.default_rng(seed)
    c = np.concatenate([b.z, b.v], -1)
    off = rng.uniform(-frac, frac, c.shape) * b.sigma
    a0 = c + off
    nx = b.z.shape[-1]
    return a0[..., :nx], a0[..., nx:], -off


@pytest.mark.parametrize("name", ["planar_quad", "chain4", "chain28"])
@pytest.mark.parametrize("fixed", [False, True])
def test_pgd_matches_oracle(gpu, orc, name, fixed):
    import torch
    import paper_2607_01203_amd as leb
    from oracle import pgd
    b = _case(name)
    if fixed:
        z0, v0, mu0 = _offcentre(b, 3)
    else:
        z0, v0, mu0 = b.z, b.v, np.zeros(b.sigma.shape)
    radius, steps, lr = 0.5, 8, 0.3
    print("case: pgd %s fixed_box=%s steps=%d" % (name, fixed, steps), flush=True)
    dyn = leb.dynamics_like(b.dyn)
    z, v, w, w0 = leb.pgd_nominal(dyn, _t(z0, gpu), _t(v0, gpu), _t(b.sigma, gpu), mu0=_t(mu0, gpu), radius=radius,
                                  steps=steps, lr=lr, fixed_box=fixed)
    torch.cuda.synchronize()
    a = np.concatenate([z.cpu().numpy(), v.cpu().numpy()], -1)
    w, w0 = w.cpu().numpy(), w0.cpu().numpy()
    a0 = np.concatenate([z0, v0], -1)
    d = orc.Dyn.like(b.dyn)
    # the start's width is the bound's width at a0 (parity tolerance of the bound, summed over rows)
    lo0, hi0, _ = orc.leb(d, z0, v0, b.sigma, mu=mu0)
    M0 = np.maximum(np.abs(lo0), np.abs(hi0)).sum(-1)
    assert (np.abs(w0 - (hi0 - lo0).sum(-1)) <= 2e-4 * M0).all()
    # the returned point lies in the search box; its width is the GPU bound's there, which
    # matches the oracle's bound at that point
    assert (np.abs(a - a0) <= radius * b.sigma * (1 + 1e-12)).all()
    mu = a0 + mu0 - a if fixed else mu0
    nx = b.z.shape[-1]
    g = leb.analytic_bound(dyn, _t(a[..., :nx], gpu), _t(a[..., nx:], gpu), _t(b.sigma, gpu), _t(mu, gpu))
    torch.cuda.synchronize()
    glo, ghi = g["r_lo"].cpu().numpy(), g["r_hi"].cpu().numpy()
    seq = np.zeros(w.shape)
    for l in range(nx):                      # the kernel's order of summation
        seq += ghi[..., l] - glo[..., l]
    np.testing.assert_array_equal(seq, w)
    lo, hi, _ = orc.leb(d, a[..., :nx], a[..., nx:], b.sigma, mu=mu)
    check_bounds(glo, ghi, lo, hi, "pgd %s" % name)
    # never wider than the start, and narrower on most units
    assert (w <= w0).all() and (w < w0).mean() >= 0.75
    # the oracle's descent from the same start: same sign decisions on most units, and
    # the same mean width within the bound's parity tolerance
    ao, wo, _ = pgd.pgd_nominal(d, z0, v0, b.sigma, mu0=mu0, radius=radius, steps=steps, lr=lr, fixed_box=fixed)
    same = (np.abs(a - ao) <= 1e-9 * b.sigma).all(-1)
    print("same path on %.3f of the units; mean width GPU %.6g oracle %.6g start %.6g"
          % (same.mean(), w.mean(), wo.mean(), w0.mean()))
    assert same.mean() >= 0.75
    assert abs(w.mean() - wo.mean()) <= 1e-3 * wo.mean()


def test_pgd_rejects_bad_arguments(gpu):
    import ctypes
    import paper_2607_01203_amd as leb
    b = _case("chain4")
    dyn = leb.dynamics_like(b.dyn)
    z0, v0, sg = _t(b.z, gpu), _t(b.v, gpu), _t(b.sigma, gpu)
    for kw in ({"radius": 1.5}, {"radius": -0.1}, {"lr": 0.0}, {"lr": float("inf")}, {"steps": -1}):
        with pytest.raises(leb.LebError):
            leb.pgd_nominal(dyn, z0, v0, sg, **kw)
    z, v, w = z0.clone(), v0.clone(), sg.new_empty(b.z.shape[:2])
    rc = leb.lib().leb_pgd_nominal(ctypes.byref(dyn), b.z.shape[0], b.z.shape[1], z0.data_ptr(), v0.data_ptr(),
                                   None, sg.data_ptr(), 2, 0.5, 1, 0.1, z.data_ptr(), v.data_ptr(), w.data_ptr(),
                                   None, None)
    assert rc == -1


def _sample_best(leb, dyn, a0, sigma, radius, K, gen, chunk):
    """Narrowest bound over K nominal points drawn uniformly from a0 +/- radius sigma
    (the travelling box), evaluated in batched launches of `chunk` candidates."""
    import torch
    nx = dyn.nx
    U = a0.shape[0] * a0.shape[1]
    best = None
    done = 0
    while done < K:
        k = min(chunk, K - done)
        u = torch.rand((k,) + tuple(a0.shape), generator=gen, dtype=torch.float64, device=a0.device)
        a = a0.unsqueeze(0) + (2.0 * u - 1.0) * radius * sigma.unsqueeze(0)
        a = a.reshape(k * a0.shape[0], a0.shape[1], -1)
        sg = sigma.unsqueeze(0).expand(k, -1, -1, -1).reshape(a.shape).contiguous()
        o = leb.analytic_bound(dyn, a[..., :nx].contiguous(), a[..., nx:].contiguous(), sg)
        w = (o["r_hi"] - o["r_lo"]).sum(-1).reshape(k, U).min(0).values
        best = w if best is None else torch.minimum(best, w)
        done += k
    return best


@pytest.mark.parametrize("name", ["planar_quad", "chain28"])
def test_pgd_beats_sampling_at_equal_time(gpu, name):
    """Per unit, the refined point's width is at most the best of as many random
    nominal points as the GPU evaluates in the time the refinement took (at
    least four per step)."""
    import torch
    import paper_2607_01203_amd as leb
    b = W.planar_quad_cfg(N=64) if name == "planar_quad" else W.chain_cfg(N=40)
    dyn = leb.dynamics_like(b.dyn)
    z0, v0, sg = _t(b.z, gpu), _t(b.v, gpu), _t(b.sigma, gpu)
    a0 = torch.cat([z0, v0], -1)
    radius, steps, lr = 1.0, 10, 0.3
    print("case: pgd vs sampling %s" % name, flush=True)
    leb.pgd_nominal(dyn, z0, v0, sg, radius=radius, steps=steps, lr=lr)
    torch.cuda.synchronize()
    t = time.perf_counter()
    z, v, w, w0 = leb.pgd_nominal(dyn, z0, v0, sg, radius=radius, steps=steps, lr=lr)
    torch.cuda.synchronize()
    t_pgd = time.perf_counter() - t
    gen = torch.Generator(device=gpu)
    gen.manual_seed(7)
    chunk = 64
    _sample_best(leb, dyn, a0, sg, radius, 2 * chunk, gen, chunk)      # warm every library call
    torch.cuda.synchronize()
    t = time.perf_counter()
    _sample_best(leb, dyn, a0, sg, radius, 8 * chunk, gen, chunk)
    torch.cuda.synchronize()
    per = (time.perf_counter() - t) / (8 * chunk)
    K = max(4 * steps, int(np.ceil(t_pgd / per)))
    best = _sample_best(leb, dyn, a0, sg, radius, K, gen, chunk)
    torch.cuda.synchronize()
    w, best, w0 = w.reshape(-1), best, w0.reshape(-1)
    print("pgd %.3f ms, %d samples; mean width start %.6g sampling %.6g pgd %.6g"
          % (t_pgd * 1e3, K, w0.mean().item(), best.mean().item(), w.mean().item()))
    assert bool((w <= best).all())


@pytest.mark.parametrize("U,few,many", [(28, 5, 600), (1, 130, 16500), (50, 3, 270), (64, 2, 300), (33, 256, 257)])
@pytest.mark.parametrize("fixed_box,steps", [(False, 3), (True, 2), (True, 0)])
def test_pgd_fused_and_by_launches_agree(gpu, U, few, many, fixed_box, steps):
    """The descent in one launch (few timesteps) and by a launch for each part
    (many): the same point and widths, bit for bit, also for a timestep with
    invalid data, a springless unit and workgroups that are not full."""
    import torch
    import paper_2607_01203_amd as leb
    b = W.chain_batch(90 + U, 1, many, U)
    z, v, sg = b.z.copy(), b.v.copy(), b.sigma.copy()
    z[0, 1, 2] = np.nan
    mu = 0.4 * sg * np.random.default_rng(U).uniform(-1.0, 1.0, sg.shape)
    dyn = leb.dynamics_like(b.dyn)
    print("case: pgd fused U=%d few=%d many=%d fixed=%s steps=%d" % (U, few, many, fixed_box, steps), flush=True)

    def run(k):
        out = leb.pgd_nominal(dyn, _t(z[:, :k], gpu), _t(v[:, :k], gpu), _t(sg[:, :k], gpu), _t(mu[:, :k], gpu),
                              radius=0.8, steps=steps, lr=0.4, fixed_box=fixed_box)
        torch.cuda.synchronize()
        return [x.cpu().numpy() for x in out]

    for x, y in zip(run(few), run(many)):
        assert np.array_equal(x, y[:, :few], equal_nan=True)
