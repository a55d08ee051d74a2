"""Timed cases of the path-guiding framework: what a renderer has it do per frame.

``listed()`` names the cases, ``draw(rng)`` gives another one of the same
ranges, ``prepare`` builds what the program holds before the call (G-buffers,
a trained state, the frame's records where a call reads them), ``run`` makes
one pass through the package's public calls, ``work`` counts the bytes and
operations a pass cannot do without and ``exact`` evaluates the same pass in
64 bits with plain torch.

Inputs follow paper_2112_09728_amd/workload.py: a value-noise height field
(normals tilted up to 35 degrees), a pinhole camera above it, roughness
U[0.05, 1], albedo U[0.2, 0.9], three spherical-Gaussian lights with random
visibility bits, a camera pan of U[-2, 2]^2 px and 2% disocclusion.  The
state is drawn with the statistics of a trained one (measured on the 1080p
pan after 32 frames: about 4.5% of the models restart per frame, so the epoch
k is 16 for nearly half of the pixels and 12 on average; pi 0.05 to 0.8 with
median 0.16, lobes of variance 5e-5 to 0.08 around the strongest light).
"""
import math

import torch

import paper_2112_09728_amd as pg

DTYPES = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
K_MAX, PI_LO, PI_HI, EPS = 16, 0.05, 0.95, 2.5e-4
F64 = torch.float64


# ------------------------------------------------------------------ the cases
def _frame(name, width, height, spp, state, first=False, image=False):
    return {"name": name, "kind": "frame", "width": width, "height": height, "spp": spp, "state": state,
            "first": first, "image": image}


def listed():
    return [
        # the smallest view (a probe or a thumbnail): three launches, latency decides
        _frame("frame_64x64_spp1_f32", 64, 64, 1, "f32"),
        # the headline: one frame of the 1080p camera pan at the paper's 1 spp
        _frame("frame_1080p_spp1_f32", 1920, 1080, 1, "f32"),
        # a 4K target with the half-precision state
        _frame("frame_4k_spp1_f16", 3840, 2160, 1, "f16"),
        # a window of odd size, BF16 state, a sample count that is no power of two
        _frame("frame_1283x717_spp3_bf16", 1283, 717, 3, "bf16"),
        # more samples per pixel (previews, offline frames), with the image they give
        _frame("frame_1080p_spp8_f32_image", 1920, 1080, 8, "f32", image=True),
        # the first frame after a camera cut: every model new, 20 picks per pixel
        _frame("first_frame_1440p_spp2_f16", 2560, 1440, 2, "f16", first=True),
        # two Gaussian lobes per pixel
        {"name": "lobes2_1080p_spp1", "kind": "lobes", "width": 1920, "height": 1080, "spp": 1, "lobes": 2},
        # positional reuse of virtual point lights under the near-field emitter
        {"name": "vpl_1080p_spp1", "kind": "vpl", "width": 1920, "height": 1080, "spp": 1, "lobes": 1},
        # gradient fit of the mixture (forward and backward) at 4K, 4 spp
        {"name": "nll_4k_spp4", "kind": "nll", "width": 3840, "height": 2160, "spp": 4},
        # the same on an odd small window, one sample per pixel
        {"name": "nll_333x241_spp1", "kind": "nll", "width": 333, "height": 241, "spp": 1},
        # densities of four given directions per pixel (other estimators' MIS weights)
        {"name": "pdf_1080p_n4_f32", "kind": "pdf", "width": 1920, "height": 1080, "n": 4, "state": "f32"},
        # a serving step: views of uneven size and sample count in one batched frame
        {"name": "batch_8_views_f16", "kind": "batch", "state": "f16",
         "views": "3840x2160x4 1280x720x8 640x360x1 1920x1080x5 2560x1440x2 1920x1080x7 640x360x3 3840x2160x1"},
    ]


def draw(rng):
    def size(most):
        """A size of log-uniform area up to `most`, odd ones as likely as even ones."""
        area = math.exp(rng.uniform(math.log(2500), math.log(most)))
        w = max(17, min(3840, round(math.sqrt(area * rng.uniform(0.7, 2.4)))))
        return w, max(9, min(2160, round(area / w)))

    kind = rng.choice(["frame"] * 5 + ["lobes", "vpl", "nll", "nll", "pdf", "batch"])
    c = {"kind": kind}
    if kind == "batch":
        views = []
        for _ in range(rng.randint(2, 8)):
            w, h = size(2_000_000)
            views.append("%dx%dx%d" % (w, h, rng.randint(1, 8)))
        return {"kind": kind, "state": rng.choice(["f16", "bf16", "f32"]), "views": " ".join(views)}
    if kind == "pdf":
        n = rng.randint(1, 8)
        c["width"], c["height"] = size(3840 * 2160 // n)
        return {**c, "n": n, "state": rng.choice(["f32", "f16", "bf16"])}
    spp = rng.choice([1, 1, 2, 3, 4, 5, 6, 7, 8])
    c["width"], c["height"] = size(3840 * 2160 if spp <= 2 else 3840 * 2160 * 2 // spp)
    c["spp"] = spp
    if kind == "frame":
        c.update(state=rng.choice(["f32", "f32", "f16", "bf16"]), first=rng.random() < 0.15,
                 image=rng.random() < 0.3)
    elif kind != "nll":
        c["lobes"] = rng.randint(1, 4) if kind == "vpl" else rng.randint(2, 4)
    return c


# ------------------------------------------------------------------ the inputs
class _Rand:
    """Seeded draws on the GPU."""

    def __init__(self, seed):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(int(seed))

    def uniform(self, lo, hi, *shape):
        return torch.rand(shape, generator=self.g, device="cuda") * (hi - lo) + lo

    def normal(self, *shape):
        return torch.randn(shape, generator=self.g, device="cuda")

    def integers(self, lo, hi, *shape):
        return torch.randint(lo, hi, shape, generator=self.g, device="cuda")


def _noise(w, h, cell, r):
    """Value noise with a quintic fade: (h, dh/dx, dh/dy) at the pixel centres."""
    nx, ny = math.ceil(w / cell) + 2, math.ceil(h / cell) + 2
    lat = r.uniform(-1.0, 1.0, ny, nx)
    xs = (torch.arange(w, device="cuda") + 0.5) / cell
    ys = (torch.arange(h, device="cuda") + 0.5) / cell
    ix, iy = xs.floor().long(), ys.floor().long()
    tx, ty = (xs - ix)[None], (ys - iy)[:, None]
    fx, fy = (t * t * t * (t * (6 * t - 15) + 10) for t in (tx, ty))
    dfx, dfy = (30 * t * t * (t - 1) ** 2 for t in (tx, ty))
    v = [[lat[(iy + j)[:, None], (ix + i)[None]] for i in (0, 1)] for j in (0, 1)]
    a = v[0][0] + (v[0][1] - v[0][0]) * fx
    b = v[1][0] + (v[1][1] - v[1][0]) * fx
    dx = ((v[0][1] - v[0][0]) * (1 - fy) + (v[1][1] - v[1][0]) * fy) * dfx / cell
    return a + (b - a) * fy, dx, (b - a) * dfy / cell


M = 4  # world texels around the window


def _scene(w, h, r, first, position=False):
    """Two consecutive windows (cur, prev) onto one world, the lights and visibility."""
    ww, wh = w + 2 * M, h + 2 * M
    z, gx, gy = (torch.zeros(wh, ww, device="cuda") for _ in range(3))
    for octave in range(3):
        vh, vx, vy = _noise(ww, wh, 32.0 * 0.5 ** octave, r)
        s = 2.5 * 0.5 ** octave
        z, gx, gy = z + s * vh, gx + s * vx, gy + s * vy
    slope = torch.sqrt(gx * gx + gy * gy)
    lim = math.tan(math.radians(35.0))
    f = torch.where(slope > lim, lim / slope.clamp(min=1e-30), torch.ones_like(slope))
    n = torch.stack([-gx * f, -gy * f, torch.ones_like(gx)])
    world = {"normal": n / n.norm(dim=0, keepdim=True), "depth": 1000.0 - z,
             "roughness": r.uniform(0.05, 1.0, wh, ww), "albedo": r.uniform(0.2, 0.9, wh, ww),
             "vis": r.integers(0, 8, wh, ww).to(torch.uint8)}
    if position:
        xs = torch.arange(ww, device="cuda") + 0.5
        ys = torch.arange(wh, device="cuda") + 0.5
        world["position"] = torch.stack([xs[None].expand(wh, ww), ys[:, None].expand(wh, ww), z])
    step = torch.round(r.uniform(-2.0, 2.0, 2) * 256) / 256
    sx, sy = (float(v) for v in step)

    def window(ox, oy):
        x0, y0 = math.floor(0.5 + ox) + M, math.floor(0.5 + oy) + M
        return {k: v[..., y0:y0 + h, x0:x0 + w].contiguous() for k, v in world.items()}

    cur, prev = window(sx, sy), window(0.0, 0.0)
    vd = torch.stack([(w / 2 - 0.5 - torch.arange(w, device="cuda"))[None].expand(h, w),
                      (h / 2 - 0.5 - torch.arange(h, device="cuda"))[:, None].expand(h, w),
                      torch.full((h, w), float(max(w, h)), device="cuda")])
    vd = (vd / vd.norm(dim=0, keepdim=True)).contiguous()
    cur["view_dir"] = prev["view_dir"] = vd
    cur["motion"] = torch.tensor([-sx, -sy], device="cuda")[:, None, None].expand(2, h, w).contiguous()
    cur["disocc"] = (r.uniform(0.0, 1.0, h, w) < 0.02).to(torch.uint8)
    if first:
        cur["motion"].zero_()
        cur["disocc"].zero_()
    u = r.uniform(0.0, 1.0, 3, 4).cpu()
    lz, phi = u[:, 0], 2 * math.pi * u[:, 1]
    ls = torch.sqrt(1 - lz * lz)
    lights = torch.stack([ls * torch.cos(phi), ls * torch.sin(phi), lz, 10 + 190 * u[:, 2], 1 + 19 * u[:, 3]], 1)
    return cur, prev, lights, 0.05


def _state(scene, lights, r, lobes, trained=None):
    """A trained state [6 lobes + 2][H][W] (FP32 values, means not offset)."""
    h, w = scene["depth"].shape
    age = torch.log(r.uniform(1e-9, 1.0, h, w)) / math.log(1 - 0.045)
    k = age.floor().clamp(0, K_MAX)
    k = torch.where(scene["roughness"] < 0.1, torch.zeros_like(k), k)
    if trained:
        k = k.clamp(min=1)
    fresh = torch.exp(-k / 4)
    planes = []
    order = torch.argsort(lights[:, 4] / lights[:, 3], descending=True)
    for j in range(lobes):
        xi = lights[order[j % 3], :3].to("cuda")
        frame = _Basis(scene["normal"].double())
        loc = frame.local([xi[c].double().expand(h, w) for c in range(3)])
        ox, oy = _to_square([loc[0], loc[1], loc[2].clamp(min=0.05)])
        start = 0.5 if lobes == 1 else 0.5 + 0.25 * (j - 0.5 * (lobes - 1))
        mx = (start * fresh + (0.5 + 0.5 * ox.float()) * (1 - fresh) + 0.04 * (1 - fresh) * r.normal(h, w))
        my = (0.5 * fresh + (0.5 + 0.5 * oy.float()) * (1 - fresh) + 0.04 * (1 - fresh) * r.normal(h, w))
        sxx = (1 / 12) * fresh + (1 - fresh) * (0.006 * torch.exp(1.0 * r.normal(h, w))).clamp(5e-5, 0.12)
        syy = (1 / 12) * fresh + (1 - fresh) * (0.008 * torch.exp(1.0 * r.normal(h, w))).clamp(5e-5, 0.12)
        rho = (-0.22 + 0.4 * r.normal(h, w)).clamp(-0.95, 0.95) * (1 - fresh)
        pi = ((0.05 + 0.17 * (1 - fresh)) * torch.exp(0.5 * (1 - fresh) * r.normal(h, w))).clamp(PI_LO, 0.9) / lobes
        planes += [mx.clamp(0.02, 0.98), my.clamp(0.02, 0.98), sxx, rho * torch.sqrt(sxx * syy), syy, pi]
    evidence = torch.where(k > 0, 1.5 * torch.exp(0.7 * r.normal(h, w)), torch.zeros_like(k))
    return torch.stack(planes + [evidence, k]).contiguous()


def _stored(g, dtype):
    """The state in its storage type (FP16 and BF16 hold the means minus 1/2)."""
    if dtype == torch.float32:
        return g.clone()
    g = g.clone()
    g[:2] -= 0.5
    return g.to(dtype)


def _values(g):
    """The FP64 values a stored state represents."""
    v = g.double()
    if g.dtype != torch.float32:
        v = v.clone()
        v[:2] += 0.5
    return v


def _inputs(case, seed):
    """Everything a pass reads, as plain tensors."""
    c = dict(case)
    r = _Rand(seed)
    kind, w, h = c["kind"], c["width"], c["height"]
    lobes = c.get("lobes", 1)
    cur, prev, lights, ambient = _scene(w, h, r, c.get("first", False), position=kind == "vpl")
    d = {"cur": cur, "prev": prev, "lights": lights, "ambient": ambient, "seed": int(seed) & 0x7FFFFFFF,
         "t": 0 if c.get("first") else int(r.integers(8, 64, 1)), "lobes": lobes, "spp": c.get("spp", 1)}
    source = cur if kind in ("nll", "pdf") else prev
    g = _state(source, lights, r, lobes, trained=kind in ("nll", "pdf"))
    d["state"] = g if kind in ("lobes", "vpl", "nll") else _stored(g, DTYPES[c["state"]])
    if kind == "vpl":
        nx, ny = math.ceil((w + 2 * M + 96) / 48), math.ceil((h + 2 * M + 96) / 48)
        sx = -48 + (torch.arange(nx, device="cuda")[None] + r.uniform(0.25, 0.75, ny, nx)) * 48
        sy = -48 + (torch.arange(ny, device="cuda")[:, None] + r.uniform(0.25, 0.75, ny, nx)) * 48
        d["lamps"] = torch.stack([sx, sy, r.uniform(3, 8, ny, nx), r.uniform(2, 30, ny, nx)], -1).contiguous()
    if kind == "nll":  # the records of a sampled and traced frame, and the parameters of the fit
        rec = _sample(d, _values(g), 1)
        rec["radiance"] = _light(d, rec)
        d["records"] = {k: v.to(torch.uint8 if k == "strategy" else torch.float32).contiguous() for k, v in rec.items()}
        l11 = torch.sqrt(g[2])
        l21 = g[3] / l11
        d["theta"] = torch.stack([g[0], g[1], l11, l21, torch.sqrt((g[4] - l21 * l21).clamp(min=1e-8)),
                                  torch.log(g[5] / (1 - g[5])), g[6], g[7]]).contiguous()
        d["grad_nll"] = r.uniform(0.5, 1.5, h, w)
    if kind == "pdf":
        v = r.normal(3, c["n"], h, w)
        v[2] = v[2].abs() * 2
        d["dirs"] = (v / v.norm(dim=0, keepdim=True)).contiguous()
    return d


def _views(case):
    """The single-view cases of a batched one."""
    out = []
    for v in case["views"].split():
        w, h, spp = (int(x) for x in v.split("x"))
        out.append({"kind": "frame", "width": w, "height": h, "spp": spp, "state": case["state"], "first": False})
    return out


def _device_frame(scene):
    f = pg.DeviceFrame.__new__(pg.DeviceFrame)
    f.view = pg.View(scene["normal"], scene["view_dir"], scene["depth"], scene["roughness"], scene["albedo"],
                     scene.get("motion"), scene.get("disocc"))
    f.vis = scene["vis"]
    f.position = scene.get("position")
    return f


BATCH_FRAME = 9


def prepare(case, seed):
    kind = case["kind"]
    if kind == "batch":
        views = [_inputs(c, seed * 31 + i) for i, c in enumerate(_views(case))]
        specs = [dict(width=d["cur"]["depth"].shape[1], height=d["cur"]["depth"].shape[0], spp=d["spp"],
                      seed=d["seed"], lights=d["lights"].numpy(), ambient=d["ambient"]) for d in views]
        guide = pg.BatchedGuide(specs, gamma_dtype=DTYPES[case["state"]])
        for i, d in enumerate(views):
            guide.gamma[i][0].copy_(d["state"])
        frames = [(_device_frame(d["cur"]), _device_frame(d["prev"])) for d in views]
        return {"kind": kind, "guide": guide, "frames": frames}
    d = _inputs(case, seed)
    w, h = case["width"], case["height"]
    cur, prev = _device_frame(d["cur"]), _device_frame(d["prev"])
    s = {"kind": kind, "cur": cur, "prev": prev, "t": d["t"], "lobes": d["lobes"]}
    if kind == "frame":
        s["image"] = case.get("image", False)
        s["guide"] = pg.Guide(w, h, d["lights"].numpy(), d["ambient"], spp=d["spp"], seed=d["seed"],
                              gamma_dtype=DTYPES[case["state"]])
    elif kind in ("lobes", "vpl"):
        s["guide"] = pg.LobesGuide(w, h, d["lights"].numpy(), d["ambient"], lobes=d["lobes"], spp=d["spp"],
                                   seed=d["seed"])
    if "guide" in s:
        s["guide"].gamma[0].copy_(d["state"])
    if kind == "vpl":
        s["ceiling"] = pg.Ceiling(dict(lamps=d["lamps"].cpu().numpy(), **CEILING))
        s["hit"] = torch.empty((d["spp"], h, w), device="cuda")
    if kind == "nll":
        rec = d["records"]
        s["samples"] = pg.Samples.wrap(rec["dir"], rec["pdf_mix"], rec["pdf_brdf"], rec["strategy"], rec["radiance"])
        s["params"] = pg.params(d["seed"], frame=d["t"])
        s["theta"] = d["theta"].requires_grad_(True)
        s["grad_nll"] = d["grad_nll"]
    if kind == "pdf":
        s["params"] = pg.params(d["seed"], frame=d["t"])
        s["state"], s["dirs"] = d["state"], d["dirs"]
    return s


def _records(s):
    return {"dir": s.dir, "pdf_mix": s.pdf_mix, "pdf_brdf": s.pdf_brdf, "strategy": s.strategy,
            "radiance": s.radiance}


def run(s):
    kind = s["kind"]
    if kind == "batch":
        g = s["guide"]
        g.cur = 0  # the frame again from the same history
        g.step(s["frames"], t=BATCH_FRAME)
        return [{"state": g.state(i), **_records(g.samples[i])} for i in range(g.n)]
    if kind == "pdf":
        return list(pg.pdf(s["params"], s["cur"].view, s["state"], s["dirs"], components=True))
    if kind == "nll":
        nll = pg.NLLFunction.apply(s["theta"], s["params"], s["cur"].view, s["samples"])
        grad, = torch.autograd.grad(nll, s["theta"], s["grad_nll"])
        return {"nll": nll, "grad": grad}
    g = s["guide"]
    g.cur = 0
    if kind == "vpl":
        p = g.params(s["t"])
        view, out = s["cur"].view, g.gamma[1]
        pg.reproject_sample_lobes(p, g.lobes, view, s["prev"].view, g.gamma[0], out, g.samples)
        pg.light_ceiling(s["ceiling"], view, s["cur"].position, g.samples, s["hit"])
        pg.em_update_vpl(p, g.lobes, view, s["cur"].position, g.samples, s["hit"], out)
        return {"state": out, "hit": s["hit"], **_records(g.samples)}
    out = {"state": g.step(s["cur"], s["prev"], frame=s["t"]), **_records(g.samples)}
    if s.get("image"):
        out["image"] = pg.estimate(g.params(s["t"]), s["cur"].view, g.samples)
    return out


def work(case):
    """Bytes: every input plane read once, every output plane written once.
    Operations: about 120 a drawn sample, 140 a training visit (own samples
    and N(k) picks, four in five of them kept), 45 a Gaussian of a lobe."""
    kind = case["kind"]
    if kind == "batch":
        parts = [work(c) for c in _views(case)]
        return {k: sum(p[k] for p in parts) for k in ("bytes", "flops")}
    px = case["width"] * case["height"]
    if kind == "pdf":
        per = {"f32": 32, "f16": 16, "bf16": 16}[case["state"]] + 28 + 24 * case["n"]
        return {"bytes": per * px, "flops": 120 * case["n"] * px}
    spp, lobes = case["spp"], case.get("lobes", 1)
    picks = 20 if case.get("first") else 8.75
    visits = 0.8 * (spp + picks)
    if kind == "nll":  # forward and backward each read the records; theta and both gradients
        return {"bytes": (2 * (21 * spp + 32 + 32) + 4 + 4 + 32) * px, "flops": 2 * 170 * visits * px}
    g = 4 * (6 * lobes + 2) if kind != "frame" else {"f32": 32, "f16": 16, "bf16": 16}[case["state"]]
    gbuffer = 12 + 12 + 4 + 4 + 4 + (0 if case.get("first") else 8 + 1 + 4 + 12) + (12 if kind == "vpl" else 1)
    per = gbuffer + (g if not case.get("first") else 0) + g + (25 + (4 if kind == "vpl" else 0)) * spp
    per += 4 if case.get("image") else 0
    return {"bytes": per * px, "flops": (120 * spp + (140 + 45 * (lobes - 1)) * visits + 150) * px}


# --------------------------------------------------------- the same in 64 bits
CEILING = {"z": 32.0, "period": 48.0, "x0": -48.0, "y0": -48.0, "ambient": 0.05}
ROUGH_MIN = float(torch.tensor(0.1))
S_D, F0 = 0.5, float(torch.tensor(0.04))
EPS32, LO32, HI32 = (float(torch.tensor(v)) for v in (EPS, PI_LO, PI_HI))


def _dot(a, b):
    return a[0] * b[0] + a[1] * b[1] + a[2] * b[2]


def _unit(v):
    inv = 1 / torch.sqrt(_dot(v, v))
    return [x * inv for x in v]


class _Basis:
    """Duff et al.'s frame around the normalised normal."""

    def __init__(self, n):
        n = _unit(list(n))
        sign = torch.where(n[2] < 0, -torch.ones_like(n[2]), torch.ones_like(n[2]))
        a = -1 / (sign + n[2])
        c = n[0] * n[1] * a
        self.t = [1 + sign * n[0] * n[0] * a, sign * c, -sign * n[0]]
        self.b = [c, sign + n[1] * n[1] * a, -n[1]]
        self.n = n

    def local(self, w):
        return [_dot(w, self.t), _dot(w, self.b), _dot(w, self.n)]

    def world(self, v):
        return [v[0] * self.t[i] + v[1] * self.b[i] + v[2] * self.n[i] for i in range(3)]


def _to_square(w):
    """M^-1: a unit direction with w_z >= 0 to the centred square [-1, 1]^2."""
    s2 = w[0] * w[0] + w[1] * w[1]
    rho = torch.sqrt(s2 / (1 + w[2]))
    big = w[0].abs() > w[1].abs()
    num, den = torch.where(big, w[1], w[0]), torch.where(big, w[0], w[1])
    t = torch.where(den != 0, num / torch.where(den != 0, den, torch.ones_like(den)), torch.zeros_like(den))
    r = torch.copysign(rho, den)
    o = r * torch.atan(t) * (4 / math.pi)
    return torch.where(big, r, o), torch.where(big, o, r)


def _to_hemisphere(ux, uy):
    a, b = 2 * ux - 1, 2 * uy - 1
    big = a.abs() > b.abs()
    r = torch.where(big, a, b)
    safe = torch.where(r != 0, r, torch.ones_like(r))
    q = torch.where(big, 0.25 * b / safe, 0.5 - 0.25 * a / safe) * math.pi
    k = r * torch.sqrt(2 - r * r)
    return [k * torch.cos(q), k * torch.sin(q), 1 - r * r]


class _Material:
    def __init__(self, scene):
        n, o = scene["normal"].double(), scene["view_dir"].double()
        self.f = _Basis(n)
        self.wo = self.f.local(_unit(list(o)))
        rough = scene["roughness"].double()
        self.a2 = rough ** 4
        self.albedo = scene["albedo"].double()
        self.valid = _dot(list(n), list(o)) > 0
        self.guided = self.valid & (rough >= ROUGH_MIN)

    def half(self, wi):
        h = _unit([self.wo[i] + wi[i] for i in range(3)])
        d = self.a2 / (math.pi * (h[0] ** 2 + h[1] ** 2 + self.a2 * h[2] ** 2) ** 2)
        return h, d, _dot(self.wo, h)

    def pdf(self, wi):
        h, d, woh = self.half(wi)
        return S_D * wi[2] / math.pi + (1 - S_D) * d * h[2] / (4 * woh)

    def g1(self, v):
        return 2 * v[2] / (v[2] + torch.sqrt(self.a2 * (v[0] ** 2 + v[1] ** 2) + v[2] ** 2))

    def value(self, wi):
        h, d, woh = self.half(wi)
        fresnel = F0 + (1 - F0) * (1 - woh) ** 5
        return self.albedo / math.pi + fresnel * d * self.g1(wi) * self.g1(self.wo) / (4 * wi[2] * self.wo[2])


class _Gauss:
    def __init__(self, g):
        self.mx, self.my = g[0], g[1]
        self.l11 = torch.sqrt((g[2] + EPS32).clamp(min=EPS32))
        self.l21 = g[3] / self.l11
        self.l22 = torch.sqrt(((g[4] + EPS32) - self.l21 ** 2).clamp(min=EPS32))

    def pdf(self, ux, uy):
        z1 = (ux - self.mx) / self.l11
        z2 = (uy - self.my - self.l21 * z1) / self.l22
        return torch.exp(-0.5 * (z1 * z1 + z2 * z2)) / (4 * math.pi ** 2 * self.l11 * self.l22)


def _philox(c0, c1, c2, c3, seed):
    """Philox4x32-10 on int64 tensors holding 32-bit words (c1 to c3 plain numbers)."""
    m = 0xFFFFFFFF
    c1, c2, c3 = (torch.full_like(c0, v & m) for v in (c1, c2, c3))
    k0, k1 = seed & m, (seed >> 32) & m
    for _ in range(10):
        p0, p1 = c0 * 0xD2511F53, c2 * 0xCD9E8D57  # the low 64 bits are right whatever the sign
        c0, c1, c2, c3 = ((p1 >> 32) & m) ^ c1 ^ k0, p1 & m, ((p0 >> 32) & m) ^ c3 ^ k1, p0 & m
        k0, k1 = (k0 + 0x9E3779B9) & m, (k1 + 0xBB67AE85) & m
    return c0, c1, c2, c3


def _pixels(h, w):
    return torch.arange(h * w, device="cuda", dtype=torch.int64).reshape(h, w)


def _reset(d, h, w):
    lobes = d["lobes"]
    out = torch.zeros(6 * lobes + 2, h, w, dtype=F64, device="cuda")
    for j in range(lobes):
        out[6 * j] = 0.5 if lobes == 1 else 0.5 + 0.25 * (j - 0.5 * (lobes - 1))
        out[6 * j + 1] = 0.5
        out[6 * j + 2] = out[6 * j + 4] = 1 / 12
        out[6 * j + 5] = LO32 / lobes
    return out


def _reproject(d, dtype):
    """The reprojected state as stored, in FP64 values."""
    cur, prev = d["cur"], d["prev"]
    h, w = cur["depth"].shape
    new = _reset(d, h, w)
    if d["t"] == 0:
        g = new
    else:
        mat = _Material(cur)
        pix = _pixels(h, w)
        fx = (pix % w).double() + 0.5 - cur["motion"][0].double()
        fy = (pix // w).double() + 0.5 - cur["motion"][1].double()
        keep = mat.guided & (cur["disocc"] == 0) & (fx >= 0) & (fy >= 0) & (fx < w) & (fy < h)
        q = (fy.clamp(0, h - 1).floor().long() * w + fx.clamp(0, w - 1).floor().long()).reshape(-1)
        zp, zq = cur["depth"], prev["depth"].reshape(-1)[q].reshape(h, w)
        nq = prev["normal"].reshape(3, -1)[:, q].reshape(3, h, w).double()
        npx = cur["normal"].double()
        g = _values(d["state"]).reshape(-1, h * w)[:, q].reshape(-1, h, w).clone()
        keep &= ~((zp - zq).abs() > 0.1 * zp) & ~(_dot(npx, nq) < 0.9) & torch.isfinite(g).all(0)
        moved = ~(npx == nq).all(0)
        fq = _Basis(nq)
        for j in range(d["lobes"]):
            lp = mat.f.local(fq.world(_to_hemisphere(g[6 * j].clamp(0, 1), g[6 * j + 1].clamp(0, 1))))
            keep &= ~(moved & (lp[2] <= 0))
            up = _unit([lp[0], lp[1], lp[2].clamp(min=1e-12)])
            ox, oy = _to_square(up)
            g[6 * j] = torch.where(moved, 0.5 + 0.5 * ox, g[6 * j])
            g[6 * j + 1] = torch.where(moved, 0.5 + 0.5 * oy, g[6 * j + 1])
        g = torch.where(keep[None], g, new)
    if dtype != torch.float32:
        g = g.clone()
        g[:2] -= 0.5
        g = _values(g.to(dtype))
    return g


def _sample(d, g, lobes):
    """The records of a frame: directions, densities and strategy codes."""
    cur, spp, t = d["cur"], d["spp"], d["t"]
    h, w = cur["depth"].shape
    mat = _Material(cur)
    active = mat.guided & (g[-1] >= 1)
    gauss = [_Gauss(g[6 * j:6 * j + 5]) for j in range(lobes)]
    wt = [torch.where(active, g[6 * j + 5], torch.zeros_like(g[0])) for j in range(lobes)]
    tot = sum(wt)
    rec = {"dir": torch.zeros(3, spp, h, w, dtype=F64, device="cuda"),
           "pdf_mix": torch.zeros(spp, h, w, dtype=F64, device="cuda"),
           "pdf_brdf": torch.zeros(spp, h, w, dtype=F64, device="cuda"),
           "strategy": torch.zeros(spp, h, w, dtype=torch.uint8, device="cuda")}
    for s in range(spp):
        zeta, xl, x1, x2 = ((v >> 8).double() * 2.0 ** -24
                            for v in _philox(_pixels(h, w), t, s, d.get("view", 0), d["seed"]))
        cs, sn = torch.cos(2 * math.pi * x2), torch.sin(2 * math.pi * x2)
        rho = torch.sqrt(-2 * torch.log1p(-x1))
        z1, z2 = rho * cs, rho * sn
        code = torch.full((h, w), 1, dtype=torch.uint8, device="cuda")
        # the BRDF's two lobes
        r = torch.sqrt(x1)
        t2 = mat.a2 * x1 / (1 - x1)
        ch = 1 / torch.sqrt(1 + t2)
        sh = torch.sqrt(t2) * ch
        hv = [sh * cs, sh * sn, ch]
        woh = _dot(mat.wo, hv)
        diffuse = xl < S_D
        cosine = [r * cs, r * sn, torch.sqrt(1 - x1)]
        l = [torch.where(diffuse, cosine[i], 2 * woh * hv[i] - mat.wo[i]) for i in range(3)]
        ok = (l[2] > 0) & (diffuse | (woh > 0))
        code = torch.where(ok, code, torch.full_like(code, 4))
        # the lobe that zeta selects
        lo = torch.zeros_like(x1)
        for j in range(lobes):
            sel = (zeta >= lo) & (zeta < lo + wt[j])
            lo = lo + wt[j]
            ux = gauss[j].mx + gauss[j].l11 * z1
            uy = gauss[j].my + gauss[j].l21 * z1 + gauss[j].l22 * z2
            inside = (ux >= 0) & (ux <= 1) & (uy >= 0) & (uy <= 1)
            v = _to_hemisphere(ux.clamp(0, 1), uy.clamp(0, 1))
            l = [torch.where(sel, v[i], l[i]) for i in range(3)]
            code = torch.where(sel, torch.where(inside, 2, 3).to(torch.uint8), code)
        code = torch.where(mat.valid, code, torch.zeros_like(code))
        live = (code == 1) | (code == 2)
        up = [l[0], l[1], l[2].clamp(min=1e-12)]
        pb = mat.pdf(up)
        ox, oy = _to_square(up)
        D = (1 - tot) * pb
        for j in range(lobes):
            D = D + wt[j] * gauss[j].pdf(0.5 + 0.5 * ox, 0.5 + 0.5 * oy)
        wd = mat.f.world(l)
        zero = torch.zeros_like(pb)
        for i in range(3):
            rec["dir"][i, s] = torch.where(live, wd[i], zero)
        rec["pdf_mix"][s] = torch.where(live, D, zero)
        rec["pdf_brdf"][s] = torch.where(live, pb, zero)
        rec["strategy"][s] = code
    return rec


def _light(d, rec):
    lights, vis = d["lights"].double(), d["cur"]["vis"]
    out = torch.zeros_like(rec["pdf_mix"])
    for s in range(d["spp"]):
        live = (rec["strategy"][s] == 1) | (rec["strategy"][s] == 2)
        w = [rec["dir"][i, s] for i in range(3)]
        L = torch.full_like(w[0], float(torch.tensor(d["ambient"])))
        for k in range(3):
            x = [float(v) for v in lights[k]]
            d2 = (w[0] - x[0]) ** 2 + (w[1] - x[1]) ** 2 + (w[2] - x[2]) ** 2
            L = L + torch.where((vis >> k) & 1 > 0, x[4] * torch.exp(-0.5 * x[3] * d2), torch.zeros_like(L))
        out[s] = torch.where(live, L, torch.zeros_like(L))
    return out


def _ceiling(d, rec):
    pos, lamps = d["cur"]["position"].double(), d["lamps"].double()
    ny, nx = lamps.shape[:2]
    rad, hit = torch.zeros_like(rec["pdf_mix"]), torch.zeros_like(rec["pdf_mix"])
    amb = float(torch.tensor(CEILING["ambient"]))
    for s in range(d["spp"]):
        live = (rec["strategy"][s] == 1) | (rec["strategy"][s] == 2)
        w = [rec["dir"][i, s] for i in range(3)]
        rises = w[2] > 0
        t = (CEILING["z"] - pos[2]) / torch.where(rises, w[2], torch.ones_like(w[2]))
        yx, yy = pos[0] + t * w[0], pos[1] + t * w[1]
        fx, fy = (yx - CEILING["x0"]) / CEILING["period"], (yy - CEILING["y0"]) / CEILING["period"]
        near = (fx >= -1) & (fx < nx + 1) & (fy >= -1) & (fy < ny + 1)
        ci, cj = fx.clamp(-2, nx + 2).floor().long(), fy.clamp(-2, ny + 2).floor().long()
        E = torch.full_like(t, amb)
        for dj in (-1, 0, 1):
            for di in (-1, 0, 1):
                i, j = ci + di, cj + dj
                ok = near & (i >= 0) & (j >= 0) & (i < nx) & (j < ny)
                lamp = lamps[j.clamp(0, ny - 1), i.clamp(0, nx - 1)]
                d2 = (yx - lamp[..., 0]) ** 2 + (yy - lamp[..., 1]) ** 2
                E = E + torch.where(ok, lamp[..., 3] * torch.exp(-d2 / (2 * lamp[..., 2] ** 2)), torch.zeros_like(E))
        inf = torch.full_like(t, math.inf)
        rad[s] = torch.where(live, torch.where(rises, E, torch.full_like(E, amb)), torch.zeros_like(E))
        hit[s] = torch.where(live, torch.where(rises, t, inf), torch.zeros_like(t))
    return rad, hit


def _training_set(d, k, rec):
    """Each member of the pixels' training sets in turn: (record planes at the
    source pixel, source index, kept)."""
    cur, spp, t = d["cur"], d["spp"], d["t"]
    h, w = cur["depth"].shape
    pix = _pixels(h, w)
    x, y = pix % w, pix // w
    kk = k.long().clamp(0, K_MAX)
    npick = 5 + (15 * (K_MAX - kk)) // K_MAX
    plane = {n: rec[n].reshape(spp, -1) for n in ("strategy", "pdf_brdf", "radiance")}
    dirs = rec["dir"].reshape(3, spp, -1)

    def member(s, q, inside):
        i = s * (h * w) + q
        st, pb = plane["strategy"].reshape(-1)[i], plane["pdf_brdf"].reshape(-1)[i].double()
        kept = inside & (st == 1) & (pb > 0)
        wd = [dirs[c].reshape(-1)[i].double() for c in range(3)]
        return wd, plane["radiance"].reshape(-1)[i].double() / torch.where(kept, pb, torch.ones_like(pb)), i, q, kept

    for s in range(spp):
        yield member(torch.full_like(pix, s), pix, torch.ones_like(pix, dtype=torch.bool))
    words = None
    for m in range(20):
        if m % 8 == 0:
            words = _philox(pix, t, (1 << 16) | (m >> 3), d.get("view", 0), d["seed"])
        word = words[(m >> 1) & 3]
        code = (((word >> 16) if m & 1 else (word & 0xFFFF)) * (48 * spp)) >> 16
        o = code // spp
        o = o + (o >= 24)
        qx, qy = x + o % 7 - 3, y + o // 7 - 3
        inside = (qx >= 0) & (qy >= 0) & (qx < w) & (qy < h) & (m < npick)
        yield member(code % spp, qy.clamp(0, h - 1) * w + qx.clamp(0, w - 1), inside)


def _train(d, g, rec, hit=None):
    """The online EM update of g in FP64."""
    cur, lobes = d["cur"], d["lobes"]
    mat = _Material(cur)
    h, w = cur["depth"].shape
    g = g.clone()
    W, k = g[6 * lobes].clone(), g[6 * lobes + 1].clone()
    gauss = [_Gauss(g[6 * j:6 * j + 5]) for j in range(lobes)]
    pis = [g[6 * j + 5].clone() for j in range(lobes)]
    rest = 1 - sum(pis)
    zero = torch.zeros(h, w, dtype=F64, device="cuda")
    B0 = zero.clone()
    sums = [[zero.clone() for _ in range(6)] for _ in range(lobes)]
    pos = cur["position"].double() if hit is not None else None
    for wd, lw, i, q, kept in _training_set(d, k, rec):
        kept = kept & mat.guided
        if hit is not None:  # towards the sample's virtual point light
            th = hit.reshape(-1)[i]
            far = ~torch.isfinite(th)
            xq = [pos[c].reshape(-1)[q] for c in range(3)]
            th = torch.where(far, torch.ones_like(th), th)
            unit = _unit([torch.where(kept, wd[c], torch.ones_like(wd[c])) for c in range(3)])
            to = [xq[c] + th * unit[c] - pos[c] for c in range(3)]
            some = _dot(to, to) > 0
            kept = kept & (far | some)
            to = _unit([torch.where(some, to[c], torch.ones_like(to[c])) for c in range(3)])
            wd = [torch.where(far, wd[c], to[c]) for c in range(3)]
        l = mat.f.local(wd)
        kept = kept & (l[2] > 0)
        l = [torch.where(kept, l[0], zero), torch.where(kept, l[1], zero), torch.where(kept, l[2], zero + 1)]
        ox, oy = _to_square(l)
        ux, uy = 0.5 + 0.5 * ox, 0.5 + 0.5 * oy
        pb = mat.pdf(l)
        wgt = torch.where(kept, lw * mat.value(l) * l[2], zero)
        ga = [pis[j] * gauss[j].pdf(ux, uy) for j in range(lobes)]
        D = rest * pb + sum(ga)
        B0 = B0 + wgt
        for j in range(lobes):
            v = wgt * ga[j] / D
            dx, dy = ux - gauss[j].mx, uy - gauss[j].my
            for c, term in enumerate((v, v * dx, v * dy, v * dx * dx, v * dx * dy, v * dy * dy)):
                sums[j][c] = sums[j][c] + term
    on = B0 > 0
    eta = 1 / (k + 1)
    sw = (1 - eta) * W + eta * B0
    safe = torch.where(on, sw, zero + 1)
    pn = []
    for j in range(lobes):
        B1 = sums[j][0]
        so, sn = (1 - eta) * pis[j] * W, eta * B1
        sg = so + sn
        fit = on & (sg > 0) & (B1 > 0)
        b, s = torch.where(fit, B1, zero + 1), torch.where(fit, sg, zero + 1)
        al, be = so / s, sn / s
        rx, ry = sums[j][1] / b, sums[j][2] / b
        sxx, sxy, syy = sums[j][3] / b - rx * rx, sums[j][4] / b - rx * ry, sums[j][5] / b - ry * ry
        old = [g[6 * j + c].clone() for c in range(5)]
        new = [old[0] + be * rx, old[1] + be * ry, al * old[2] + be * sxx + al * be * rx * rx,
               al * old[3] + be * sxy + al * be * rx * ry, al * old[4] + be * syy + al * be * ry * ry]
        for c in range(5):
            g[6 * j + c] = torch.where(fit, new[c], old[c])
        pn.append(sg / safe)
    if lobes == 1 and not d.get("lobe_clamp"):
        pn = [pn[0].clamp(LO32, HI32)]
    else:
        pn = [p.clamp(min=LO32 * 0.25 / lobes) for p in pn]
        tt = sum(pn)
        pn = [p * tt.clamp(LO32, HI32) / tt for p in pn]
    for j in range(lobes):
        g[6 * j + 5] = torch.where(on, pn[j], pis[j])
    g[6 * lobes] = torch.where(on, sw, W)
    g[6 * lobes + 1] = torch.where(on, (k + 1).clamp(max=K_MAX), k)
    return g


def _image(d, rec):
    mat = _Material(d["cur"])
    acc = torch.zeros_like(mat.a2)
    for s in range(d["spp"]):
        l = mat.f.local([rec["dir"][i, s] for i in range(3)])
        D = rec["pdf_mix"][s]
        live = ((rec["strategy"][s] == 1) | (rec["strategy"][s] == 2)) & (D > 0) & (l[2] > 0)
        l = [torch.where(live, l[0], acc * 0), torch.where(live, l[1], acc * 0), torch.where(live, l[2], acc * 0 + 1)]
        v = mat.value(l) * rec["radiance"][s] * l[2] / torch.where(live, D, torch.ones_like(D))
        acc = acc + torch.where(live, v, torch.zeros_like(v))
    return torch.where(mat.valid, acc / d["spp"], torch.zeros_like(acc))


def _exact_view(case, d):
    dtype = DTYPES[case.get("state", "f32")]
    g = _reproject(d, dtype)
    rec = _sample(d, g, d["lobes"])
    hit = None
    if case["kind"] == "vpl":
        rec["radiance"], hit = _ceiling(d, rec)
    else:
        rec["radiance"] = _light(d, rec)
    g = _train(d, g, rec, hit)
    if dtype != torch.float32:
        g[:2] -= 0.5
    out = {"state": g, **rec, "strategy": None}
    if hit is not None:
        out["hit"] = hit
    if case.get("image"):
        out["image"] = _image(d, rec)
    return out


def exact(case, seed):
    kind = case["kind"]
    if kind == "batch":
        out = []
        for i, c in enumerate(_views(case)):
            d = _inputs(c, seed * 31 + i)
            d["t"], d["view"] = BATCH_FRAME, i
            out.append(_exact_view(c, d))
        return out
    d = _inputs(case, seed)
    if kind == "pdf":
        mat, g = _Material(d["cur"]), _values(d["state"])
        gauss = _Gauss(g)
        pe = torch.where(mat.guided & (g[7] >= 1), g[5], torch.zeros_like(g[5]))
        out = [[], [], []]
        for j in range(case["n"]):
            l = mat.f.local(_unit([d["dirs"][c, j].double() for c in range(3)]))
            up = mat.valid & (l[2] > 0)
            l = [l[0], l[1], torch.where(up, l[2], torch.ones_like(l[2]))]
            ox, oy = _to_square(l)
            zero = torch.zeros_like(pe)
            pgd = torch.where(up, gauss.pdf(0.5 + 0.5 * ox, 0.5 + 0.5 * oy), zero)
            pb = torch.where(up, mat.pdf(l), zero)
            for o, v in zip(out, (pe * pgd + (1 - pe) * pb, pgd, pb)):
                o.append(v)
        return [torch.stack(o) for o in out]
    if kind == "nll":
        return _exact_nll(d)
    d["lobe_clamp"] = kind in ("lobes", "vpl")
    return _exact_view(case, d)


def _exact_nll(d):
    th = d["theta"].detach().double()
    mat = _Material(d["cur"])
    l11, l21, l22 = th[2], th[3], th[4]
    A, B, C = l11 ** 2 + EPS32, l11 * l21, l21 ** 2 + l22 ** 2 + EPS32
    gauss = _Gauss(torch.stack([th[0], th[1], l11 ** 2, B, l21 ** 2 + l22 ** 2]))
    pi = torch.sigmoid(th[5])
    det = A * C - B * B
    ia, ib, ic = C / det, -B / det, A / det
    zero = torch.zeros_like(pi)
    loss, gm, gs, gl = zero, [zero, zero], [zero, zero, zero], zero
    for wd, lw, _, _, kept in _training_set(d, th[7], d["records"]):
        l = mat.f.local(wd)
        kept = kept & mat.guided & (l[2] > 0)
        l = [torch.where(kept, l[0], zero), torch.where(kept, l[1], zero), torch.where(kept, l[2], zero + 1)]
        ox, oy = _to_square(l)
        ux, uy = 0.5 + 0.5 * ox, 0.5 + 0.5 * oy
        ga = pi * gauss.pdf(ux, uy)
        D = ga + (1 - pi) * mat.pdf(l)
        wgt = torch.where(kept, lw * mat.value(l) * l[2], zero)
        gam = ga / D
        dx, dy = ux - th[0], uy - th[1]
        vx, vy = ia * dx + ib * dy, ib * dx + ic * dy
        loss = loss - wgt * torch.log(D)
        wg = wgt * gam
        gm = [gm[0] - wg * vx, gm[1] - wg * vy]
        gs = [gs[0] - 0.5 * wg * (vx * vx - ia), gs[1] - 0.5 * wg * (vx * vy - ib), gs[2] - 0.5 * wg * (vy * vy - ic)]
        gl = gl - wgt * (gam - pi)
    sc = d["grad_nll"].double()
    grad = torch.stack([gm[0], gm[1], 2 * (gs[0] * l11 + gs[1] * l21), 2 * (gs[1] * l11 + gs[2] * l21),
                        2 * gs[2] * l22, gl, zero, zero]) * sc
    return {"nll": loss, "grad": grad}
