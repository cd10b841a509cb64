"""GPU CROWN + Theorem 2 bound (leb_nn_bound) against the NN oracle: the
16-256-256-256-12 workload, other widths and depths, ragged chunks, stable
boxes, off-centre boxes, bad inputs and 10^6-sample soundness."""
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


def _run(leb, net, z, v, sg, dev, mu=None, zonotope=False):
    import torch
    mlp = leb.MLP(net.W, net.b, net.nx, True)
    out = leb.nn_bound(mlp, _t(z, dev), _t(v, dev), _t(sg, dev), None if mu is None else _t(mu, dev),
                       zonotope=zonotope)
    torch.cuda.synchronize()
    res = {k: x.cpu().numpy() for k, x in out.items()}
    mlp.close()
    return res


def _oracle(net, z, v, sg, mu=None):
    from oracle import nn
    a = np.concatenate([z, v], -1)
    return nn.leb(net.W, net.b, a, sg, mu=mu)


def test_nn_small_slice_parity(gpu):
    import paper_2607_01203_amd as leb
    b = W.nn_cfg()
    z, v, sg = b.z[:2, :7], b.v[:2, :7], b.sigma[:2, :7]
    print("case: nn 16-256x3-12, 14 boxes", flush=True)
    g = _run(leb, b.net, z, v, sg, gpu)
    o = _oracle(b.net, z, v, sg)
    print("worst", check_bounds(g["r_lo"], g["r_hi"], o["r_lo"], o["r_hi"], "nn small"))
    assert (g["flags"] == 0).all()


def test_nn_full_config_sampled(gpu):
    """64 trajectories x 50 steps (3200 boxes, one chunk of work): oracle on a sample."""
    import paper_2607_01203_amd as leb
    b = W.nn_cfg()
    print("case: nn full 64x50", flush=True)
    g = _run(leb, b.net, b.z, b.v, b.sigma, gpu, zonotope=True)
    idx = np.random.default_rng(0).choice(3200, 120, replace=False)
    bt, kt = idx // 50, idx % 50
    o = _oracle(b.net, b.z[bt, kt], b.v[bt, kt], b.sigma[bt, kt])
    print("worst", check_bounds(g["r_lo"][bt, kt], g["r_hi"][bt, kt], o["r_lo"], o["r_hi"], "nn full"))
    assert (g["c_bar"] - g["rho_bar"] <= g["r_lo"]).all() and (g["c_bar"] + g["rho_bar"] >= g["r_hi"]).all()


@pytest.mark.parametrize("widths,nx", [([16, 128, 128, 128, 12], 12), ([32, 64, 64, 8], 8), ([16, 48, 16], 16)])
def test_nn_other_shapes(gpu, widths, nx):
    import paper_2607_01203_amd as leb
    rng = W.rng_for(77)
    Wl, bl = W.mlp_weights(rng, widths)
    net = W.MLPNet(Wl, bl, nx, widths[0] - nx, True)
    a = rng.uniform(-1, 1, (3, 5, widths[0]))
    sg = rng.uniform(0.005, 0.05, (3, 5, widths[0]))
    print("case: nn widths %s" % widths, flush=True)
    g = _run(leb, net, a[..., :nx].copy(), a[..., nx:].copy(), sg, gpu)
    o = _oracle(net, a[..., :nx], a[..., nx:], sg)
    check_bounds(g["r_lo"], g["r_hi"], o["r_lo"], o["r_hi"], "widths %s" % widths)


def test_nn_stable_offcentre_and_bad(gpu):
    import paper_2607_01203_amd as leb
    b = W.nn_cfg()
    z, v = b.z[:1, :6].copy(), b.v[:1, :6].copy()
    sg = b.sigma[:1, :6].copy()
    sg[0, 0] = 1e-9                                    # stable box: bound ~ [0, 0]
    mu = np.random.default_rng(1).uniform(-0.02, 0.02, sg.shape)
    mu[0, 0] = 0.0
    z[0, 5, 3] = np.nan                                # invalid data
    print("case: nn stable / off-centre / bad", flush=True)
    g = _run(leb, b.net, z, v, sg, gpu, mu=mu)
    o = _oracle(b.net, z[:, :5], v[:, :5], sg[:, :5], mu=mu[:, :5])
    check_bounds(g["r_lo"][:, :5], g["r_hi"][:, :5], o["c_lo"], o["c_hi"], "nn off-centre")
    assert np.abs(g["r_hi"][0, 0]).max() < 1e-9 and np.abs(g["r_lo"][0, 0]).max() < 1e-9
    assert np.isinf(g["r_lo"][0, 5]).all() and g["flags"][0, 5] & 2


def test_nn_soundness_1e6(gpu):
    import paper_2607_01203_amd as leb
    from oracle import nn
    b = W.nn_cfg()
    z, v, sg = b.z[:8], b.v[:8], b.sigma[:8]          # 400 boxes x 2500 samples
    print("case: nn 1e6 samples", flush=True)
    g = _run(leb, b.net, z, v, sg, gpu)
    a = np.concatenate([z, v], -1).reshape(-1, 16)
    c, rho = nn.box_of(a, sg.reshape(-1, 16))
    rng = W.rng_for(1_000_001)
    lo = g["r_lo"].reshape(-1, 12)
    hi = g["r_hi"].reshape(-1, 12)
    viol = 0
    for s in range(0, 400, 50):
        pts = W.sample_box_points(rng, (c - rho)[s:s + 50], (c + rho)[s:s + 50], 2500)
        r, eps = nn.remainder(b.net.W, b.net.b, a[s:s + 50], pts)
        viol += int(((r > hi[s:s + 50, None] + eps) | (r < lo[s:s + 50, None] - eps)).sum())
    assert viol == 0


def test_nn_bound_two_chunks(gpu):
    """4,300 boxes: two chunks of the bound's work buffers (4,096 boxes at
    most), the second ragged; the oracle on boxes at both ends of each."""
    import paper_2607_01203_amd as leb
    rng = W.rng_for(78)
    Wl, bl = W.mlp_weights(rng, [16, 32, 32, 12])
    net = W.MLPNet(Wl, bl, 12, 4, True)
    a = rng.uniform(-1, 1, (1, 4300, 16))
    sg = rng.uniform(0.005, 0.1, (1, 4300, 16))
    print("case: nn bound 4300 boxes", flush=True)
    g = _run(leb, net, a[..., :12].copy(), a[..., 12:].copy(), sg, gpu)
    idx = np.array([0, 1, 4095, 4096, 4097, 4299])
    o = _oracle(net, a[0, idx, :12], a[0, idx, 12:], sg[0, idx])
    check_bounds(g["r_lo"][0, idx], g["r_hi"][0, idx], o["r_lo"], o["r_hi"], "two chunks")


@pytest.mark.parametrize("widths", [[16, 16, 16, 16, 4], [16, 48, 80, 112, 12], [16, 256, 240, 32, 12],
                                    [16, 64, 256, 256, 16, 8], [16, 256, 12]])
@pytest.mark.parametrize("shift", [0.0, 50.0, -50.0])
def test_nn_hidden_targets_tiles(gpu, widths, shift):
    """The 16-input hidden-layer passes: fewer tiles than waves, a ragged last
    row block, the widest layers, a fourth hidden layer above them, and layers
    whose neurons are mixed, all stably active or all stably inactive."""
    rng = W.rng_for(910 + widths[1] + len(widths))
    Wl, bl = W.mlp_weights(rng, widths)
    bl = [x + np.float32(shift) if 0 < i < len(bl) - 1 else x for i, x in enumerate(bl)]
    net = W.MLPNet(Wl, bl, 12, 4, False)
    import paper_2607_01203_amd as leb
    a = rng.uniform(-1, 1, (2, 4, 16))
    sg = rng.uniform(0.005, 0.3, (2, 4, 16))
    print("case: nn hidden targets %s shift %g" % (widths, shift), flush=True)
    import torch
    mlp = leb.MLP(net.W, net.b, 12, False)
    out = leb.nn_bound(mlp, _t(a[..., :12], gpu), _t(a[..., 12:], gpu), _t(sg, gpu))
    torch.cuda.synchronize()
    o = _oracle(net, a[..., :12], a[..., 12:], sg)
    lo, hi = out["r_lo"].cpu().numpy(), out["r_hi"].cpu().numpy()
    # a constant network over a box that crosses layer-1 kinks: the oracle's bound is
    # exactly 0, the kernel's is its rounding allowance, 2^-40 times a few sums of
    # magnitudes, each at most the chain |b| + |W| m
    zero = (o["r_lo"] == 0.0) & (o["r_hi"] == 0.0)
    m = np.abs(a) + 2.0 * sg
    for w, x in zip(net.W, net.b):
        m = m @ np.abs(np.asarray(w, np.float64)).T + np.abs(np.asarray(x, np.float64))
    assert (lo[zero] <= 0.0).all() and (hi[zero] >= 0.0).all()
    assert (np.maximum(-lo, hi)[zero] <= 8.0 * 2.0 ** -40 * m[zero]).all()
    check_bounds(lo[~zero], hi[~zero], o["r_lo"][~zero], o["r_hi"][~zero], "hidden targets")
    mlp.close()


@pytest.mark.parametrize("widths", [[32, 256, 240, 12], [48, 16, 32, 16, 48, 8], [240, 96, 20], [32, 32, 64, 256, 64]])
@pytest.mark.parametrize("shift", [0.0, 50.0, -50.0])
def test_nn_chain_tiles(gpu, widths, shift):
    """The chain of a target layer over listed neurons and columns: inputs wider
    than a tile, none to sixteen listed tiles, every slicing of the k-steps, ragged
    outputs, layers mixed, all stably active or all stably inactive."""
    import torch
    import paper_2607_01203_amd as leb
    rng = W.rng_for(1210 + widths[1] + len(widths))
    Wl, bl = W.mlp_weights(rng, widths)
    bl = [x + np.float32(shift) if 0 < i < len(bl) - 1 else x for i, x in enumerate(bl)]
    nx = widths[0] - 4
    a = rng.uniform(-1, 1, (2, 3, widths[0]))
    sg = rng.uniform(0.005, 0.1, (2, 3, widths[0]))
    print("case: nn chain %s shift %g" % (widths, shift), flush=True)
    mlp = leb.MLP(Wl, bl, nx, False)
    out = leb.nn_bound(mlp, _t(a[..., :nx], gpu), _t(a[..., nx:], gpu), _t(sg, gpu))
    torch.cuda.synchronize()
    o = _oracle(W.MLPNet(Wl, bl, nx, 4, False), a[..., :nx], a[..., nx:], sg)
    lo, hi = out["r_lo"].cpu().numpy(), out["r_hi"].cpu().numpy()
    # rows whose exact bound is 0 (a constant network): the rounding allowance, as above
    zero = (o["r_lo"] == 0.0) & (o["r_hi"] == 0.0)
    m = np.abs(a) + 2.0 * sg
    for w, x in zip(Wl, bl):
        m = m @ np.abs(np.asarray(w, np.float64)).T + np.abs(np.asarray(x, np.float64))
    assert (lo[zero] <= 0.0).all() and (hi[zero] >= 0.0).all()
    assert (np.maximum(-lo, hi)[zero] <= 8.0 * 2.0 ** -40 * m[zero]).all()
    check_bounds(lo[~zero], hi[~zero], o["r_lo"][~zero], o["r_hi"][~zero], "nn chain")
    mlp.close()


@pytest.mark.parametrize("widths", [[16, 256, 256, 256, 12], [32, 48, 144, 64], [16, 16, 20], [48, 128, 16, 33]])
def test_nn_groups_of_boxes(gpu, widths):
    """From 1,024 boxes on, 16 boxes share a workgroup in the forward pass and the
    relaxations: the same bits as a box alone, in every place of a ragged last
    group, with an invalid box among them."""
    import torch
    import paper_2607_01203_amd as leb
    rng = W.rng_for(1510 + widths[1] + len(widths))
    Wl, bl = W.mlp_weights(rng, widths)
    nx = widths[0] - 4
    a = rng.uniform(-1, 1, (1, 1033, widths[0]))
    sg = rng.uniform(0.0, 0.1, a.shape)
    mu = sg * rng.uniform(-1.2, 1.2, a.shape)
    a[0, 700, 1] = np.nan
    print("case: nn groups %s" % widths, flush=True)
    mlp = leb.MLP(Wl, bl, nx, False)

    def run(sl):
        out = leb.nn_bound(mlp, _t(a[:, sl, :nx], gpu), _t(a[:, sl, nx:], gpu), _t(sg[:, sl], gpu), _t(mu[:, sl], gpu))
        torch.cuda.synchronize()
        return [out[k].cpu().numpy() for k in ("r_lo", "r_hi", "flags")]

    big = run(slice(0, 1033))
    for s0, s1 in ((0, 40), (690, 710), (1020, 1033)):
        for x, y in zip(big, run(slice(s0, s1))):
            assert np.array_equal(x[:, s0:s1], y)
    mlp.close()
