"""The first-bounce estimator the guided samples feed: per pixel the mean of
f_r L cos / D over its samples (null samples count zero).

Parity of pg_estimate with the oracle on the same records, and the point of
the method on the analytic light field: on the 1080p camera-pan sequence the
1-spp estimate with guided sampling against BRDF sampling alone (pi held at
0), relative MSE against an FP64 reference integral (mixture of BRDF and
light-lobe sampling, 2048 samples per pixel) on 32768 random guided pixels at
four frames, by roughness class."""
import sys

import numpy as np
import pytest
import torch

import oracle as O
import paper_2112_09728_amd as pg
from paper_2112_09728_amd import workload as wl
from pgtest import paired_ratio_ci, dev, gpu_view, host, random_gamma, records_host, rel_err

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


def say(*a):
    print(*a, file=sys.stderr, flush=True)


@pytest.mark.parametrize("W,H,spp", [(67, 45, 4), (130, 33, 1)])
def test_estimate_parity(W, H, spp):
    say(f"case: estimate {W}x{H} spp {spp}")
    seed = 7100 + W + spp
    scene = wl.make_scene(W, H, seed)
    g = random_gamma(H, W, np.random.default_rng(seed))
    p, P = pg.params(seed, frame=5), O.params(seed, frame=5)
    view = gpu_view(scene)
    s = pg.Samples(spp, H, W)
    pg.sample_mis(p, view, dev(g), s)
    pg.light_field(pg.lights_struct(scene["lights"], float(scene["ambient"])), view, dev(scene["vis"]), s)
    est = host(pg.estimate(p, view, s))
    torch.cuda.synchronize()
    eo = O.estimate(P, O.OView(scene), records_host(s))
    pos = eo > 0
    assert (est[~pos] == 0).all()
    r = rel_err(est[pos], eo[pos])
    say(f"  rel err max {r.max():.2e} q99.9 {np.quantile(r, 0.999):.2e} median {np.median(r):.2e}")
    assert np.quantile(r, 0.999) <= 1e-5 and r.max() <= 1e-3


def test_guided_estimator_against_brdf_sampling():
    cfg = wl.CONFIGS["1080p_spp1_64f_fp32_pan"]
    W, H, seed = 1920, 1080, cfg["seed"]
    frames, evals, n_px, n_ref = 32, (7, 15, 23, 31), 32768, 2048
    say(f"case: estimator study, 1080p pan, frames {evals}, {n_px} px, reference {n_ref} samples")
    seq = wl.Sequence(W, H, seed)
    fr = seq.frame(0)
    lights, amb = fr["lights"], float(fr["ambient"])
    guided = pg.Guide(W, H, lights, amb, spp=1, seed=seed)
    brdf = pg.Guide(W, H, lights, amb, spp=1, seed=seed, pi_init=0.0, pi_lo=0.0, pi_hi=0.0)
    rng = np.random.default_rng(seed)
    classes = [(0.1, 0.3), (0.3, 0.6), (0.6, 1.01)]
    acc = {c: {"g": 0.0, "b": 0.0, "ref2": 0.0, "n": 0, "se2": 0.0} for c in classes}
    pairs_g, pairs_b = [], []
    prev = None
    for t in range(frames):
        if t:
            fr = seq.frame(t)
        cur = pg.DeviceFrame(fr)
        guided.step(cur, prev, frame=t)
        brdf.step(cur, prev, frame=t)
        prev = cur
        if t not in evals:
            continue
        pg_ = guided.params(t)
        eg = host(pg.estimate(pg_, cur.view, guided.samples))
        eb = host(pg.estimate(brdf.params(t), cur.view, brdf.samples))
        torch.cuda.synchronize()
        rough = fr["roughness"]
        valid = (np.einsum("chw,chw->hw", fr["normal"], fr["view_dir"]) > 0) & (rough >= 0.1)
        cand = np.flatnonzero(valid.reshape(-1))
        px = np.sort(rng.choice(cand, size=n_px, replace=False))
        ref, se = O.reference(O.params(seed, frame=t), O.OView(fr), lights, amb, fr["vis"], px, n_ref)
        r = rough.reshape(-1)[px]
        pairs_g.append((eg.reshape(-1)[px] - ref) ** 2 / (ref ** 2).sum())
        pairs_b.append((eb.reshape(-1)[px] - ref) ** 2 / (ref ** 2).sum())
        for c in classes:
            m = (r >= c[0]) & (r < c[1])
            a = acc[c]
            a["g"] += float(((eg.reshape(-1)[px][m] - ref[m]) ** 2).sum())
            a["b"] += float(((eb.reshape(-1)[px][m] - ref[m]) ** 2).sum())
            a["ref2"] += float((ref[m] ** 2).sum())
            a["se2"] += float((se[m] ** 2).sum())
            a["n"] += int(m.sum())
    say("  roughness class | pixels | rel. MSE BRDF only | rel. MSE guided | ratio | reference SE^2 / MSE")
    tot = {"g": 0.0, "b": 0.0, "ref2": 0.0, "se2": 0.0}
    for c in classes:
        a = acc[c]
        say(f"  [{c[0]:.1f}, {c[1]:.1f}) | {a['n']} | {a['b'] / a['ref2']:.4f} | {a['g'] / a['ref2']:.4f} | "
            f"{a['g'] / a['b']:.3f} | {a['se2'] / a['g']:.1e}")
        for k in tot:
            tot[k] += a[k]
    ratio = tot["g"] / tot["b"]
    say(f"  all | {sum(acc[c]['n'] for c in classes)} | {tot['b'] / tot['ref2']:.4f} | "
        f"{tot['g'] / tot['ref2']:.4f} | {ratio:.3f} | {tot['se2'] / tot['g']:.1e}")
    assert tot["se2"] < 0.05 * tot["g"]  # the reference is far more accurate than either estimate
    rr, lo, hi = paired_ratio_ci(np.concatenate(pairs_g), np.concatenate(pairs_b))
    say(f"  guided / BRDF-only MSE over the evaluated frames: {rr:.3f}, paired bootstrap 95% [{lo:.3f}, {hi:.3f}]")
    assert ratio < 1.0


@pytest.mark.parametrize("spp", [1, 3, 8])
def test_estimate_of_records_that_are_not_finite(spp):
    """A record that counts (a BRDF or guided draw with a density) and holds a
    NaN direction, radiance or infinity shows in its pixel's estimate; one that
    does not count changes nothing, whatever it holds."""
    W, H, seed = 67, 19, 7300 + spp
    scene = wl.make_scene(W, H, seed)
    rng = np.random.default_rng(seed)
    p, view = pg.params(seed, frame=5), gpu_view(scene)
    s = pg.Samples(spp, H, W)
    pg.sample_mis(p, view, dev(random_gamma(H, W, rng)), s)
    pg.light_field(pg.lights_struct(scene["lights"], float(scene["ambient"])), view, dev(scene["vis"]), s)
    clean = host(pg.estimate(p, view, s))
    code, D = host(s.strategy), host(s.pdf_mix)
    live = ((code == 1) | (code == 2)) & (D > 0)
    pick = rng.random((spp, H, W)) < 0.1
    d, L = host(s.dir).copy(), host(s.radiance).copy()
    what = rng.integers(0, 3, (spp, H, W))
    d[:, pick & (what == 0)] = np.nan
    L[pick & (what == 1)] = np.nan
    L[pick & (what == 2)] = np.inf
    s.dir.copy_(dev(d))
    s.radiance.copy_(dev(L))
    got = host(pg.estimate(p, view, s))
    bad = (pick & live).any(0)
    assert bad.sum() > 50 and (pick & ~live).any()
    assert not np.isfinite(got[bad]).any()
    assert (got[~bad] == clean[~bad]).all()
