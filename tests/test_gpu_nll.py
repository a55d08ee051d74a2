"""The radiance-weighted NLL of the mixture and its hand-written adjoint on the
GPU: parity with the oracle, central differences in FP64, and a gradient fit
through torch.autograd against batch EM on the same samples."""
import sys

import numpy as np
import pytest
import torch

import oracle as O
import paper_2112_09728_amd as pg
from paper_2112_09728_amd import workload as wl
from pgtest import dev, gpu_view, host, random_gamma, records_host

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


def say(*a):
    print(*a, file=sys.stderr, flush=True)


def _setup(W, H, spp, seed):
    """Frame-0 records (every model new: BRDF samples, N(0) = 20 picks)."""
    scene = wl.make_scene(W, H, seed)
    p = pg.params(seed, frame=0)
    view = gpu_view(scene)
    g0 = torch.zeros((8, H, W), dtype=torch.float32, device="cuda")
    s = pg.Samples(spp, H, W)
    pg.reproject_sample(p, view, None, None, g0, s)
    pg.light_field(pg.lights_struct(scene["lights"], float(scene["ambient"])), view,
                   dev(scene["vis"]), s)
    torch.cuda.synchronize()
    return scene, view, s, host(g0)


def _theta(H, W, rng):
    return np.stack([rng.uniform(0.3, 0.7, (H, W)), rng.uniform(0.3, 0.7, (H, W)),
                     rng.uniform(0.05, 0.2, (H, W)), rng.uniform(-0.05, 0.05, (H, W)),
                     rng.uniform(0.05, 0.2, (H, W)), rng.uniform(-2, 2, (H, W)),
                     np.zeros((H, W)), np.zeros((H, W))]).astype(np.float32)


@pytest.mark.parametrize("W,H,spp", [(64, 48, 4), (37, 29, 1)])
def test_nll_and_adjoint_match_oracle(W, H, spp):
    say(f"case: nll {W}x{H} spp {spp}")
    seed = 9000 + W + spp
    scene, view, s, _ = _setup(W, H, spp, seed)
    th = _theta(H, W, np.random.default_rng(seed))
    go = np.random.default_rng(seed + 1).uniform(0.5, 2.0, (H, W)).astype(np.float32)
    p = pg.params(seed, frame=0)
    nll, grad = pg.nll_backward(p, view, s, dev(th), grad_out=dev(go))
    torch.cuda.synchronize()
    P = O.params(seed, frame=0)
    nll_o, grad_o = O.nll(P, O.OView(scene), records_host(s), th, grad_out=go)
    nll_g, grad_g = host(nll), host(grad)
    scale_n = np.abs(nll_o).max() + 1e-30
    en = np.abs(nll_g - nll_o) / (np.abs(nll_o) + 1e-3 * scale_n)
    say(f"  nll rel err max {en.max():.2e}")
    assert en.max() <= 1e-4
    for c in range(6):
        sc = np.abs(grad_o[c]).max() + 1e-30
        e = np.abs(grad_g[c] - grad_o[c]) / (np.abs(grad_o[c]) + 1e-3 * sc)
        say(f"  grad[{c}] rel err max {e.max():.2e} p99 {np.quantile(e, 0.99):.2e}")
        assert np.quantile(e, 0.99) <= 1e-4 and e.max() <= 1e-3, c
    assert (grad_g[6:] == 0).all()


def test_adjoint_against_fp64_central_differences_on_crop():
    """Central differences of the FP64 oracle's NLL (h = 1e-4) on a 32x32
    crop against the GPU adjoint."""
    say("case: adjoint vs FD 32x32 crop")
    W = H = 96
    seed = wl.SEED_BASE + 4
    scene, view, s, _ = _setup(W, H, 4, seed)
    th = _theta(H, W, np.random.default_rng(seed))
    p = pg.params(seed, frame=0)
    _, grad = pg.nll_backward(p, view, s, dev(th))
    torch.cuda.synchronize()
    grad_g = host(grad)
    P = O.params(seed, frame=0)
    ov = O.OView(scene)
    rec = records_host(s)
    rect = (32, 32, 64, 64)
    h = 1e-4
    x0, y0, x1, y1 = rect
    for c in range(6):
        tp, tm = th.astype(np.float64), th.astype(np.float64)
        tp = tp.copy()
        tm = tm.copy()
        tp[c] += h
        tm[c] -= h
        fd = (O.nll(P, ov, rec, tp, rect=rect)[0] - O.nll(P, ov, rec, tm, rect=rect)[0]) / (2 * h)
        fd = fd[y0:y1, x0:x1]
        gg = grad_g[c, y0:y1, x0:x1]
        sc = np.abs(fd).max() + 1e-30
        e = np.abs(gg - fd) / (np.abs(fd) + 1e-2 * sc)
        say(f"  channel {c}: rel err p99 {np.quantile(e, 0.99):.2e} max {e.max():.2e}")
        assert np.quantile(e, 0.99) <= 1e-4 and e.max() <= 1e-3, c


def test_gradient_fit_reaches_batch_em_likelihood():
    """Adam on (mu, Cholesky factor, logit pi) through NLLFunction against 16
    iterations of batch EM on the same samples, both without the pi clamp: the
    fit must reach (or beat) EM's summed NLL within 1%."""
    say("case: gradient fit vs batch EM")
    W, H, spp = 64, 64, 4
    seed = wl.SEED_BASE + 4
    scene, view, s, g0 = _setup(W, H, spp, seed)
    p = pg.params(seed, frame=0, flags=pg.PG_NO_CLAMP | pg.PG_EM_BATCH)
    ge = dev(g0)
    pg.em_update(p, view, s, ge, iterations=16)
    gem = host(ge)
    l11 = np.sqrt(np.maximum(gem[2], 0))
    l21 = np.where(l11 > 0, gem[3] / np.where(l11 > 0, l11, 1), 0)
    l22 = np.sqrt(np.maximum(gem[4] - l21 ** 2, 0))
    pi = np.clip(gem[5], 1e-6, 1 - 1e-6)
    th_em = np.stack([gem[0], gem[1], l11, l21, l22, np.log(pi / (1 - pi)), gem[6], gem[7]])
    pn = pg.params(seed, frame=0, flags=pg.PG_NO_CLAMP)
    nll_em, _ = pg.nll_backward(pn, view, s, dev(th_em.astype(np.float32)), want_grad=False)
    # gradient fit from the new-model state
    th0 = np.stack([g0[0], g0[1], np.sqrt(g0[2]), g0[3], np.sqrt(g0[4]),
                    np.log(g0[5] / (1 - g0[5])), g0[6], g0[7]]).astype(np.float32)
    theta = torch.tensor(th0, device="cuda", requires_grad=True)
    opt = torch.optim.Adam([theta], lr=0.02)
    mask = torch.zeros_like(theta)
    mask[:6] = 1
    hist = []
    for it in range(300):
        opt.zero_grad()
        loss = pg.NLLFunction.apply(theta, pn, view, s).sum()
        loss.backward()
        theta.grad.mul_(mask)
        opt.step()
        hist.append(float(loss.detach()))
    torch.cuda.synchronize()
    total_em = float(nll_em.sum())
    assert np.isfinite(total_em)
    say(f"  summed NLL: EM(16) {total_em:.2f}  gradient fit start {hist[0]:.2f} end {hist[-1]:.2f}")
    assert hist[-1] < hist[0]
    assert hist[-1] <= total_em + 0.01 * abs(total_em)


@pytest.mark.parametrize("W,H,spp", [(1, 1, 1), (33, 9, 2), (31, 17, 3), (17, 16, 4), (45, 33, 5), (70, 19, 8)])
def test_nll_of_trained_records_at_tile_edges(W, H, spp):
    """Remainders of the training tile (32x8 up to spp 3, 16x16 above), lists of
    every length (k 0 to 16, records of a guided frame), the loss and the
    gradient each on its own, and pixels that train nothing; the bounds are
    those of the frame-0 comparison above."""
    say(f"case: nll tile edges {W}x{H} spp {spp}")
    seed = 9100 + W + spp
    scene = wl.make_scene(W, H, seed)
    rng = np.random.default_rng(seed)
    p = pg.params(seed, frame=3)
    view = gpu_view(scene)
    s = pg.Samples(spp, H, W)
    pg.sample_mis(p, view, dev(random_gamma(H, W, rng, k_lo=0)), s)
    pg.light_field(pg.lights_struct(scene["lights"], float(scene["ambient"])), view, dev(scene["vis"]), s)
    th = _theta(H, W, rng)
    th[7] = rng.integers(0, 17, (H, W))
    go = rng.uniform(0.5, 2.0, (H, W)).astype(np.float32)
    nll, grad = pg.nll_backward(p, view, s, dev(th), grad_out=dev(go))
    loss_only, _ = pg.nll_backward(p, view, s, dev(th), want_grad=False)
    _, grad_only = pg.nll_backward(p, view, s, dev(th), grad_out=dev(go), want_nll=False)
    torch.cuda.synchronize()
    nll_o, grad_o = O.nll(O.params(seed, frame=3), O.OView(scene), records_host(s), th, grad_out=go)
    idle = (scene["roughness"] < np.float32(0.1))
    for n, g in ((host(nll), host(grad)), (host(loss_only), host(grad_only))):
        en = np.abs(n - nll_o) / (np.abs(nll_o) + 1e-3 * (np.abs(nll_o).max() + 1e-30))
        assert en.max() <= 1e-4
        for c in range(6):
            e = np.abs(g[c] - grad_o[c]) / (np.abs(grad_o[c]) + 1e-3 * (np.abs(grad_o[c]).max() + 1e-30))
            assert np.quantile(e, 0.99) <= 1e-4 and e.max() <= 1e-3, c
        assert (g[6:] == 0).all() and (n[idle] == 0).all() and (g[:, idle] == 0).all()


@pytest.mark.parametrize("spp", [1, 4])
def test_nll_where_only_a_far_gaussian_is_left(spp):
    """A weight pi that rounds to 1 (logit 100) leaves the Gaussian alone, and
    every sample 10 to 14.3 standard deviations from it: densities down to
    exp(-102), below FP32's normal numbers.  The loss and its gradient stay
    those of the Gaussian (posterior 1).  Bounds: u carries up to 4 ulp (2.4e-7)
    and the deviation z = |u - mu| / 0.034 up to 14.3, so z^2 / 2 (50 and more)
    is off by 1e-4 at most, 2e-6 of the loss; the weight's BRDF adds 1e-5."""
    say(f"case: nll of far samples, spp {spp}")
    W, H = 45, 19
    one = np.ones((H, W), np.float32)
    scene = dict(normal=np.stack([0 * one, 0 * one, one]), view_dir=np.stack([0 * one, 0.6 * one, 0.8 * one]),
                 depth=one, roughness=0.5 * one, albedo=0.5 * one)
    t, b = O.onb(np.array([[0.0, 0.0, 1.0]]))
    u = np.array([[0.12, 0.15]])
    l = O.sq2hemi(u)[0]
    w = l[0] * t[0] + l[1] * b[0] + l[2] * np.array([0.0, 0.0, 1.0])
    rec = dict(dir=np.broadcast_to(w.astype(np.float32)[:, None, None, None], (3, spp, H, W)).copy(),
               pdf_mix=np.full((spp, H, W), 0.3, np.float32), pdf_brdf=np.full((spp, H, W), 0.3, np.float32),
               strategy=np.ones((spp, H, W), np.uint8), radiance=np.full((spp, H, W), 2.0, np.float32))
    z = np.linspace(10.0, 14.3, W * H).reshape(H, W)
    sd, ang = np.sqrt(0.03 ** 2 + 2.5e-4), np.linspace(0.1, 1.4, W)[None, :]
    th = np.stack([u[0, 0] + z * sd * np.cos(ang), u[0, 1] + z * sd * np.sin(ang), 0.03 * one, 0 * one, 0.03 * one,
                   100 * one, 0 * one, 16 * one]).astype(np.float32)
    p = pg.params(7, frame=2)
    s = pg.Samples.wrap(*(dev(rec[k]) for k in ("dir", "pdf_mix", "pdf_brdf", "strategy", "radiance")))
    view = gpu_view(scene)
    nll, grad = pg.nll_backward(p, view, s, dev(th))
    loss_only, _ = pg.nll_backward(p, view, s, dev(th), want_grad=False)
    _, grad_only = pg.nll_backward(p, view, s, dev(th), want_nll=False)
    torch.cuda.synchronize()
    nll_o, grad_o = O.nll(O.params(7, frame=2), O.OView(scene), rec, th)
    assert np.isfinite(nll_o).all() and nll_o.min() > 0
    for n, g in ((host(nll), host(grad)), (host(loss_only), host(grad_only))):
        assert np.isfinite(n).all() and np.isfinite(g).all()
        assert (np.abs(n - nll_o) <= 2e-5 * nll_o).all()
        for c in range(5):
            assert (np.abs(g[c] - grad_o[c]) <= 2e-5 * (np.abs(grad_o[c]) + 1e-3 * np.abs(grad_o[c]).max())).all(), c
        assert (g[5] == 0).all()


@pytest.mark.parametrize("spp", [1, 3, 4, 8])
def test_nll_tile_shapes_bitwise_identical(spp):
    """Every tile that pg_nll_backward takes gives the same bits, the loss and the
    gradient together and each on its own (the default is 32x8 up to 3 spp and at
    7 and 8, 16x16 between); the others are refused: the records of all planes,
    the lists and the pick table must fit 64 KiB, although two passes from 4 spp
    would need less."""
    say(f"case: nll tile invariance, spp {spp}")
    W, H, seed = 99, 61, 6100 + spp
    scene = wl.make_scene(W, H, seed)
    rng = np.random.default_rng(seed)
    view = gpu_view(scene)
    p0 = pg.params(seed, frame=3)
    s = pg.Samples(spp, H, W)
    pg.sample_mis(p0, view, dev(random_gamma(H, W, rng, k_lo=0)), s)
    pg.light_field(pg.lights_struct(scene["lights"], float(scene["ambient"])), view, dev(scene["vis"]), s)
    th = _theta(H, W, rng)
    th[7] = rng.integers(0, 17, (H, W))
    th, go = dev(th), dev(rng.uniform(0.5, 2.0, (H, W)).astype(np.float32))
    nll0, grad0 = pg.nll_backward(p0, view, s, th, grad_out=go)
    assert torch.isfinite(nll0).all() and (grad0[:6].abs().amax((1, 2)) > 0).all()
    for tw, th_ in pg.guide.TILES:
        say(f"  tile {tw}x{th_}")
        p = pg.params(seed, frame=3, tile_w=tw, tile_h=th_)
        lds = (tw + 6) * (th_ + 6) * spp * 16 + (spp + 20) * tw * th_ * 2 + ((96 * spp + 15) & ~15)
        if lds > 64 * 1024:
            with pytest.raises(RuntimeError, match="LDS"):
                pg.nll_backward(p, view, s, th, grad_out=go)
            continue
        nll, grad = pg.nll_backward(p, view, s, th, grad_out=go)
        loss_only, _ = pg.nll_backward(p, view, s, th, want_grad=False)
        _, grad_only = pg.nll_backward(p, view, s, th, grad_out=go, want_nll=False)
        torch.cuda.synchronize()
        assert torch.equal(nll, nll0) and torch.equal(loss_only, nll0), (tw, th_)
        assert torch.equal(grad, grad0) and torch.equal(grad_only, grad0), (tw, th_)


def test_nll_next_to_the_largest_number():
    """A pixel whose loss, 2.5e38 to 3.3e38, is a number in FP32 (the same record
    everywhere, the weight scaled to reach it) keeps it: sums are formed in
    natural logarithms, not in units that overflow before they do."""
    say("case: nll next to FP32's largest number")
    W, H = 45, 9
    one = np.ones((H, W), np.float32)
    scene = dict(normal=np.stack([0 * one, 0 * one, one]), view_dir=np.stack([0 * one, 0.6 * one, 0.8 * one]),
                 depth=one, roughness=0.5 * one, albedo=0.5 * one)
    w = O.sq2hemi(np.array([[0.42, 0.55]]))[0].astype(np.float32)
    th = np.stack([0.8 * one, 0.8 * one, 0.05 * one, 0 * one, 0.05 * one, -2 * one, 0 * one, 16 * one]).astype(np.float32)
    rec = dict(dir=np.broadcast_to(w[:, None, None, None], (3, 1, H, W)).copy(),
               pdf_mix=np.full((1, H, W), 0.3, np.float32), pdf_brdf=np.full((1, H, W), 0.3, np.float32),
               strategy=np.ones((1, H, W), np.uint8), radiance=np.ones((1, H, W), np.float32))
    P, ov = O.params(7, frame=2), O.OView(scene)
    base, _ = O.nll(P, ov, rec, th)
    # interior pixels have the same six members (own and five picks)
    top = base.max()
    assert top > 0
    rec["radiance"][:] = (3.3e38 / top * 0.999)
    nll_o, _ = O.nll(P, ov, rec, th)
    s = pg.Samples.wrap(*(dev(rec[k]) for k in ("dir", "pdf_mix", "pdf_brdf", "strategy", "radiance")))
    nll, _ = pg.nll_backward(pg.params(7, frame=2), gpu_view(scene), s, dev(th), want_grad=False)
    torch.cuda.synchronize()
    n = host(nll)
    big = nll_o > 2.5e38
    assert big.sum() > 50
    assert (np.abs(n - nll_o) <= 2e-5 * nll_o).all()
