"""Performance cases of the light-field library: what its users have it do,
through the public functions of ``paper_1903_03837_amd``.

listed()  the named cases;   draw(rng)  one more case of the same ranges;
prepare() a case's inputs on the GPU, from the seed alone;   run()  one pass;
work()    the bytes and operations a pass cannot do without;
exact()   the pass's outputs in 64 bits, written here in plain torch.

Scenes are seeded stand-ins for CT data: nested-ellipsoid phantoms in stored
Hounsfield units (u16) and Gaussian blobs (u8, f32) in the box [-1, 1]^3 under
piecewise-linear transfer functions, on the sphere of radius sqrt(3).
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_1903_03837_amd as lp

R = math.sqrt(3.0)
DEV = "cuda"
TORCH_DTYPE = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}


# --------------------------------------------------------------------------
# the cases
# --------------------------------------------------------------------------
def listed():
    return [
        # the point set and nearest-point queries of one small set: the
        # smallest call (a program mapping a batch of hit points to texels)
        dict(name="points_query", kind="points", n=2048, nq=65537, K=5),
        # a real-time viewer: both eyes of one frame from the paper's storage
        # configuration (upper hemisphere of 12288 origins, 23576 directions, FP16)
        dict(name="lookup_stereo", kind="lookup", M=12288, N=23576, rows=6144, dtype="f16", views=2, W=1280, H=720,
             K=5, nn=False),
        # view synthesis in bulk: 32 full-HD views of the CT-like field
        dict(name="lookup_bulk", kind="lookup", M=2048, N=2048, rows=0, dtype="f32", views=32, W=1920, H=1080, K=5,
             nn=False),
        # views of the largest field a GPU is given (12.9 GB)
        dict(name="lookup_wide", kind="lookup", M=32768, N=32768, rows=0, dtype="f32", views=8, W=1920, H=1080, K=5,
             nn=False),
        # fitting a field to images: views, loss gradient and its transpose
        dict(name="lookup_l2", kind="l2", M=2048, N=2048, rows=0, dtype="f32", views=32, W=1920, H=1080, K=5),
        # a small preview field (u8 volume, latency)
        dict(name="generate_small", kind="generate", vol=64, vtype="u8", M=256, N=256, rows=0, spp=16, bounces=4,
             g=0.0, light="directional", grid=4, dtype="f32", surface=False, waves=0),
        # one shard of the highest-resolution field: 2048 of 32768 origin rows
        dict(name="generate_fine", kind="shard", vol=512, M=32768, N=32768, begin=15360, end=17408, spp=16, bounces=8,
             g=0.3, grid=8, dtype="f32", waves=3),
        # the isosurface variant (what the paper renders)
        dict(name="generate_surface", kind="generate", vol=256, vtype="u16", M=1024, N=1024, rows=0, spp=16, bounces=4,
             g=0.0, light="area", grid=8, dtype="f32", surface=True, waves=0),
        # ground-truth views for the evaluation of a field
        dict(name="render_views", kind="render", vol=256, views=4, W=480, H=270, spp=256, bounces=8, g=0.3, grid=5),
        # the whole differentiable step on the CT-like workload: field with
        # kept samples, views + loss + transpose, path-replay adjoint
        dict(name="ct_step", kind="step", vol=256, M=2048, N=2048, spp=64, bounces=8, g=0.3, grid=5, views=32, W=1920,
             H=1080, K=5),
        # a transfer function fitted to a target field: every ray carries an
        # adjoint, through autograd, nothing kept from the forward
        dict(name="train_field", kind="train", vol=128, N=1024, spp=32, bounces=4, grid=8, keep=False),
        # the image metrics of an evaluation, full-HD pairs
        dict(name="metrics", kind="metrics", n=2, W=1920, H=1080),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["points", "lookup", "lookup", "l2", "generate", "generate", "shard", "render", "step", "train",
                       "metrics"])
    dtype = rng.choice(["f32", "f16", "bf16"])
    if kind == "points":
        return dict(kind=kind, n=_log(rng, 200, 65535), nq=_log(rng, 5000, 2000000), K=rng.choice([1, 3, 5, 9]))
    if kind in ("lookup", "l2"):
        M = _log(rng, 256, 12288)
        N = M if rng.random() < 0.6 else _log(rng, 256, 23576)
        rows = M // 2 if rng.random() < 0.3 else 0
        views = rng.choice([1, 2, 4, 8])
        W = _log(rng, 160, 1920)
        c = dict(kind=kind, M=M, N=N, rows=rows, dtype=dtype, views=views, W=W, H=max(11, W * 9 // 16),
                 K=rng.choice([1, 3, 5, 5, 5, 9]))
        if kind == "lookup":
            c["nn"] = rng.random() < 0.2
        return c
    if kind == "generate":
        surface = rng.random() < 0.3
        N = _log(rng, 128, 1500)
        M = N if rng.random() < 0.7 else _log(rng, 128, 1500)
        return dict(kind=kind, vol=8 * rng.randint(4, 32), vtype=rng.choice(["u8", "u16", "f32"]), M=M, N=N,
                    rows=M // 2 if rng.random() < 0.3 else 0, spp=_log(rng, 4, 64), bounces=rng.choice([1, 2, 4, 8]),
                    g=rng.choice([0.0, 0.3, 0.6]), light=rng.choice(["directional", "area"]),
                    grid=rng.choice([0, 4, 5, 8, 11]), dtype=dtype, surface=surface, waves=rng.choice([0, 0, 3, 4]))
    if kind == "shard":
        N = _log(rng, 4096, 24000)
        count = min(N // 2, int(2.0e7 / N))
        begin = rng.randint(0, N - count)
        return dict(kind=kind, vol=rng.choice([256, 512]), M=N, N=N, begin=begin, end=begin + count,
                    spp=rng.choice([4, 16]), bounces=8, g=0.3, grid=8, dtype=dtype, waves=rng.choice([0, 3]))
    if kind == "render":
        W = _log(rng, 64, 640)
        return dict(kind=kind, vol=8 * rng.randint(8, 32), views=rng.randint(1, 4), W=W, H=max(8, W * 3 // 4),
                    spp=_log(rng, 8, 256), bounces=8, g=0.3, grid=rng.choice([4, 5, 8]))
    if kind == "step":
        W = _log(rng, 160, 1280)
        return dict(kind=kind, vol=8 * rng.randint(12, 32), M=_log(rng, 256, 1500), N=_log(rng, 256, 1500),
                    spp=rng.choice([8, 16, 33, 64]), bounces=8, g=0.3, grid=rng.choice([5, 8]),
                    views=rng.choice([2, 8]), W=W, H=W * 9 // 16, K=rng.choice([1, 5]))
    if kind == "train":
        return dict(kind=kind, vol=8 * rng.randint(6, 20), N=_log(rng, 100, 800), spp=rng.choice([8, 16, 32]),
                    bounces=4, grid=rng.choice([4, 8]), keep=rng.random() < 0.5)
    W = _log(rng, 96, 1280)
    return dict(kind=kind, n=rng.randint(1, 4), W=W, H=max(64, W * 9 // 16 + rng.randint(0, 8)))


# --------------------------------------------------------------------------
# inputs
# --------------------------------------------------------------------------
def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(seed)


def _rotation(rng):
    q, r = np.linalg.qr(rng.standard_normal((3, 3)))
    q = q * np.sign(np.diag(r))
    return q if np.linalg.det(q) > 0 else q * np.array([1.0, 1.0, -1.0])


def _unit(rng):
    v = rng.standard_normal(3)
    return v / np.linalg.norm(v)


def _quadric(n, c, rot, a, z):
    """sum_k ((rot_k . (p - c)) / a_k)^2 at the voxel centres of slices z."""
    i = torch.arange(n, device=DEV, dtype=torch.float32) + 0.5
    x, y = (i - float(c[0]))[None, None, :], (i - float(c[1]))[None, :, None]
    w = (z.float() + 0.5 - float(c[2]))[:, None, None]
    q = 0.0
    for k in range(3):
        s = 1.0 / float(a[k])
        q = q + ((float(rot[k, 0]) * s) * x + (float(rot[k, 1]) * s) * y + (float(rot[k, 2]) * s) * w) ** 2
    return q


def _phantom(n, seed, bricked):
    """u16 CT-like phantom: nested ellipsoids, background -1000 HU, noise of 20 HU, stored HU + 1024."""
    rng = np.random.default_rng(seed)
    half = n / 2.0
    c0 = np.full(3, half) + rng.uniform(-0.05, 0.05, 3) * n
    ells = [(c0, _rotation(rng), rng.uniform(0.6, 0.95, 3) * (half - np.abs(c0 - half).max()), rng.uniform(-100, 300))]
    for _ in range(11 if n <= 256 else 39):
        pc, _, pa, _ = ells[rng.integers(len(ells))]
        a = rng.uniform(0.5, 0.9, 3) * pa.min()
        off = _unit(rng) * (pa.min() - a.max()) * rng.uniform() ** (1.0 / 3.0)
        ells.append((pc + off, _rotation(rng), a, rng.uniform(-1000.0, 2000.0)))
    g = _gen(seed)
    out = torch.empty((n, n, n), dtype=torch.int16, device=DEV)
    for z0 in range(0, n, 64):
        z = torch.arange(z0, min(n, z0 + 64), device=DEV)
        hu = torch.full((len(z), n, n), -1000.0, device=DEV)
        for c, rot, a, h in ells:
            if z0 - a.max() <= c[2] <= z0 + 64 + a.max():
                hu = torch.where(_quadric(n, c, rot, a, z) <= 1.0, h, hu)
        hu += torch.randn(hu.shape, generator=g, device=DEV) * 20.0
        out[z0:z0 + len(z)] = (hu + 1024.0).round_().clamp_(0.0, 32767.0).to(torch.int16)
    if bricked:
        b = n // 8
        out = out.view(b, 8, b, 8, b, 8).permute(0, 2, 4, 1, 3, 5).contiguous()
    return lp.Volume(out.reshape(-1), (n, n, n), 24.0, 3024.0, brick=8 if bricked else 0)


def _blobs(n, seed, vtype):
    """Sum of eight anisotropic Gaussian blobs, largest value 1 (f32) or 255 (u8)."""
    rng = np.random.default_rng(seed)
    v = torch.zeros((n, n, n), device=DEV)
    z = torch.arange(n, device=DEV)
    for _ in range(8):
        q = _quadric(n, rng.uniform(0.2 * n, 0.8 * n, 3), _rotation(rng), rng.uniform(3.0, 12.0, 3) * n / 64.0, z)
        v += float(rng.uniform(0.5, 1.0)) * torch.exp(-0.5 * q)
    v /= v.max()
    if vtype == "u8":
        return lp.Volume((v * 255.0).round().to(torch.uint8).reshape(-1), (n, n, n), 0.0, 255.0)
    return lp.Volume(v.reshape(-1), (n, n, n), 0.0, 1.0)


def _volume(case, seed, bricked=False):
    vtype = case.get("vtype", "u16")
    return _phantom(case["vol"], seed, bricked) if vtype == "u16" else _blobs(case["vol"], seed, vtype)


def _medium(seed, opaque_colours=False):
    """256-entry table through six knots, transparent at the first, density scale 10."""
    rng = np.random.default_rng(seed + 1)
    pos = np.concatenate([[0.0], np.sort(rng.uniform(0.0, 1.0, 4)), [1.0]])
    val = rng.uniform(0.0, 1.0, (6, 4))
    val[0, 3] = 0.0
    if opaque_colours:
        val[:, :3] = 0.2 + 0.7 * val[:, :3]
    s = np.arange(256) / 255.0
    lut = np.stack([np.interp(s, pos, val[:, c]) for c in range(4)], -1).astype(np.float32)
    return lp.Medium(torch.from_numpy(lut).to(DEV), 10.0)


def _light(kind, seed):
    rng = np.random.default_rng(seed + 2)
    u = _unit(rng)
    if kind == "directional":
        return lp.Light(kind=0, dir=tuple(u))
    t1 = np.cross(u, [0.0, 0.0, 1.0] if abs(u[2]) < 0.9 else [1.0, 0.0, 0.0])
    t1 /= np.linalg.norm(t1)
    t2 = np.cross(t1, u)
    return lp.Light(kind=1, corner=tuple(2.0 * R * u - 0.5 * R * (t1 + t2)), e1=tuple(R * t1), e2=tuple(R * t2),
                    radiance=(4.0, 4.0, 4.0))


def _cameras(count, seed):
    rng = np.random.default_rng(seed + 3)
    out = []
    for _ in range(count):
        d, dist = _unit(rng), rng.uniform(2.5, 4.0) * R
        up = (0.0, 0.0, 1.0) if abs(d[2]) < 0.99 else (1.0, 0.0, 0.0)
        out.append(lp.Camera(tuple(dist * d), (0.0, 0.0, 0.0), up, 2.0 * math.asin(R / dist) * 1.05))
    return out


def _params(case, seed):
    surface = bool(case.get("surface", False))
    return lp.GenParams(M=case.get("M", case.get("N", 1)), N=case.get("N", 1), radius=R, spp=case.get("spp", 16),
                        max_bounces=case.get("bounces", 4), g=case.get("g", 0.0), seed=4000 + seed,
                        origin_rows=case.get("rows", 0), grid=case.get("grid", 0), surface=int(surface),
                        iso=(0.35 if case.get("vtype") == "f32" else 90.0 if case.get("vtype") == "u8" else 524.0)
                        if surface else 0.0,
                        row_begin=case.get("begin", 0), row_end=case.get("end", 0),
                        waves_per_simd=case.get("waves", 0))


def _field(case, seed):
    p = _params(case, seed)
    g = _gen(seed + 4)
    lf = torch.empty((p.rows, p.N, 3), dtype=TORCH_DTYPE[case["dtype"]], device=DEV)
    return lf.uniform_(0.0, 1.0, generator=g), p


def prepare(case, seed):
    kind, s = case["kind"], dict(case=case)
    if kind == "points":
        q = torch.randn((case["nq"], 3), generator=_gen(seed), device=DEV)
        s["query"] = q / q.norm(dim=1, keepdim=True)
    elif kind in ("lookup", "l2"):
        s["lf"], s["prm"] = _field(case, seed)
        s["cams"] = _cameras(case["views"], seed)
        if kind == "l2":
            s["target"] = torch.rand((case["views"], case["H"], case["W"], 3), generator=_gen(seed + 5), device=DEV)
    elif kind == "metrics":
        # a path-traced-like view (smooth, in [0, 1]) and a noisy version of it
        shape = (case["n"], case["H"], case["W"], 3)
        g = _gen(seed)
        x = torch.linspace(0.0, 1.0, case["W"], device=DEV)[None, None, :, None]
        y = torch.linspace(0.0, 1.0, case["H"], device=DEV)[None, :, None, None]
        f = torch.rand((4, case["n"], 1, 1, 3), generator=g, device=DEV) * 20.0 + 2.0
        a = 0.5 + 0.25 * torch.sin(f[0] * x + f[1] * y) + 0.2 * torch.sin(f[2] * x * y + f[3])
        s["a"] = (a + 0.02 * torch.randn(shape, generator=g, device=DEV)).contiguous()
        s["b"] = (a + 0.05 * torch.randn(shape, generator=g, device=DEV)).contiguous()
    else:
        s["vol"] = _volume(case, seed, bricked=kind == "shard")
        s["med"] = _medium(seed, opaque_colours=bool(case.get("surface", False)))
        s["light"] = _light("directional" if kind == "train" else case.get("light", "area"), seed)
        s["prm"] = _params(dict(case, vtype="f32") if kind == "train" else case, seed)
        if kind == "train":
            s["vol"] = _blobs(case["vol"], seed, "f32")
            s["target"] = torch.rand((case["N"], case["N"], 3), generator=_gen(seed + 5), device=DEV) * 0.3
            s["scale"] = torch.tensor(s["med"].scale)
        if kind == "shard":
            s["out"] = torch.zeros((case["M"], case["N"], 3), dtype=TORCH_DTYPE[case["dtype"]], device=DEV)
        if kind in ("render", "step"):
            s["cams"] = _cameras(case["views"], seed)
        if kind == "step":
            s["target"] = torch.rand((case["views"], case["H"], case["W"], 3), generator=_gen(seed + 5), device=DEV) * 0.3
            s["srad"] = torch.empty((case["M"], case["N"], case["spp"], 3), device=DEV)
    return s


# --------------------------------------------------------------------------
# one pass
# --------------------------------------------------------------------------
def run(s):
    c = s["case"]
    kind = c["kind"]
    if kind == "points":
        return lp.points(c["n"], s["query"], c["K"])
    if kind == "lookup":
        return lp.lookup(s["lf"], s["prm"], s["cams"], c["W"], c["H"], c["K"], with_nn=c["nn"])
    if kind == "l2":
        return lp.lookup_l2(s["lf"], s["prm"], s["cams"], s["target"], c["K"])
    if kind == "generate":
        return lp.generate(s["vol"], s["med"], s["light"], s["prm"], dtype=c["dtype"])
    if kind == "shard":
        lp.generate(s["vol"], s["med"], s["light"], s["prm"], dtype=c["dtype"], out=s["out"])
        return s["out"][c["begin"]:c["end"]]
    if kind == "render":
        return lp.render_views(s["vol"], s["med"], s["light"], s["prm"], s["cams"], c["W"], c["H"])
    if kind == "step":
        lf = lp.generate(s["vol"], s["med"], s["light"], s["prm"], sample_radiance=s["srad"])
        img, d_lf = lp.lookup_l2(lf, s["prm"], s["cams"], s["target"], c["K"])
        d_lut, d_scale = lp.generate_backward(s["vol"], s["med"], s["light"], s["prm"], d_lf,
                                              sample_radiance=s["srad"])
        return lf, img, d_lf, d_lut, d_scale
    if kind == "train":
        lut = s["med"].lut.detach().requires_grad_(True)
        scale = s["scale"].detach().requires_grad_(True)
        lf = lp.LightFieldFn.apply(lut, scale, s["vol"], s["light"], s["prm"], c["keep"])
        loss = 0.5 * (lf - s["target"]).square().sum()
        d_lut, d_scale = torch.autograd.grad(loss, (lut, scale))
        return lf.detach(), d_lut, d_scale
    a, b = s["a"], s["b"]
    return lp.ssim(a, b, 1.0), lp.cw_ssim(a, b, 1.0)


# --------------------------------------------------------------------------
# what a pass cannot do without
# --------------------------------------------------------------------------
# Operations of one traced sample of a ray that meets the box: two tentative
# points (position, trilinear value, classification, decision: 40 each; one
# random block of 60; two logarithms).  Of all rays of the sphere about two
# thirds meet the box.  A nearest-point search takes about 150 operations and
# a blended texel 6.
_SAMPLE = 2.0 / 3.0 * (2 * 40 + 60 + 8)
_SEARCH, _TEXEL = 150.0, 6.0


def work(case):
    kind = case["kind"]
    item = {"f32": 4, "f16": 2, "bf16": 2}[case.get("dtype", "f32")]
    if kind == "points":
        n, nq, K = case["n"], case["nq"], case["K"]
        return {"bytes": 12.0 * n + 12.0 * nq + 8.0 * nq * K, "flops": _SEARCH * nq}
    if kind in ("lookup", "l2"):
        px = float(case["views"] * case["W"] * case["H"])
        texels = px * case["K"] ** 2
        # (a field larger than the views is read in part: about one texel per pixel)
        field = 3.0 * item * min((case["rows"] or case["M"]) * case["N"], px)
        if kind == "lookup":
            return {"bytes": field + px * (12 + (8 if case["nn"] else 0)),
                    "flops": px * 2 * _SEARCH + texels * _TEXEL}
        return {"bytes": field + 12.0 * (case["rows"] or case["M"]) * case["N"] + 24.0 * px,
                "flops": px * 2 * _SEARCH + 2 * texels * _TEXEL}
    if kind == "metrics":
        px = float(case["n"] * case["W"] * case["H"])
        # two images of three channels: one transform forward, eight back, by
        # 5 n log2 n each; the windowed moments and indices of both metrics
        return {"bytes": 24.0 * px, "flops": px * 6 * (9 * 5 * math.log2(case["W"] * case["H"]) + 8 * 12 + 60)}
    vol = float(case["vol"]) ** 3 * {"u8": 1, "u16": 2, "f32": 4}["f32" if kind == "train" else case.get("vtype", "u16")]
    if kind == "render":
        px = float(case["views"] * case["W"] * case["H"])
        return {"bytes": vol + 12.0 * px, "flops": px * case["spp"] * _SAMPLE}
    if kind == "shard":
        rays = float((case["end"] - case["begin"]) * case["N"])
        return {"bytes": vol + 3.0 * item * rays, "flops": rays * case["spp"] * _SAMPLE}
    if kind == "generate":
        rays = float((case["rows"] or case["M"]) * case["N"])
        return {"bytes": vol + 3.0 * item * rays, "flops": rays * case["spp"] * _SAMPLE}
    if kind == "step":
        rays, px = float(case["M"] * case["N"]), float(case["views"] * case["W"] * case["H"])
        texels = px * case["K"] ** 2
        return {"bytes": 2 * vol + rays * (12.0 * case["spp"] + 24.0) + 24.0 * px,
                "flops": rays * case["spp"] * _SAMPLE + px * 2 * _SEARCH + 2 * texels * _TEXEL}
    rays = float(case["N"]) ** 2
    return {"bytes": 2 * vol + 36.0 * rays, "flops": 3 * rays * case["spp"] * _SAMPLE}


# --------------------------------------------------------------------------
# the same in 64 bits
# --------------------------------------------------------------------------
F64, I64 = torch.float64, torch.int64
PHI_M1 = (math.sqrt(5.0) - 1.0) / 2.0
FIB = [0, 1]
while len(FIB) < 26:
    FIB.append(FIB[-1] + FIB[-2])


def _sf_points(n):
    i = torch.arange(n, device=DEV, dtype=F64)
    phi = 2.0 * math.pi * torch.frac(i * PHI_M1)
    z = 1.0 - (2.0 * i + 1.0) / n
    st = torch.sqrt((1.0 - z) * (1.0 + z))
    return torch.stack([torch.cos(phi) * st, torch.sin(phi) * st, z], -1)


def _nearest(pts, q, K):
    """Indices [nq, K] (-1: none) and squared chords of the K nearest lattice neighbours of q (unit, 64 bits)."""
    n = pts.shape[0]
    fib = torch.tensor(FIB, device=DEV)
    z = q[:, 2]
    arg = n * math.pi * math.sqrt(5.0) * (1.0 - z * z)
    k = torch.floor(torch.log(arg.clamp_min(1e-30)) / math.log((1.0 + PHI_M1) ** 2)).clamp(2, 20).to(I64)
    f0, f1 = fib[k], fib[k + 1]
    wrap = lambda f: 2.0 * math.pi * (f * PHI_M1 - torch.round(f * PHI_M1))  # noqa: E731
    b00, b01, b10, b11 = wrap(f0.double()), wrap(f1.double()), -2.0 * f0 / n, -2.0 * f1 / n
    det = b00 * b11 - b01 * b10
    phi, zz = torch.atan2(q[:, 1], q[:, 0]), z - (1.0 - 1.0 / n)
    c0, c1 = torch.floor((b11 * phi - b01 * zz) / det), torch.floor((b00 * zz - b10 * phi) / det)
    chord = lambda i: (pts[i] - q[:, None]).square().sum(-1)  # noqa: E731
    corner = torch.stack([b10 * (c0 + (s & 1)) + b11 * (c1 + (s >> 1)) + 1.0 - 1.0 / n for s in range(4)], -1)
    corner = corner.clamp(-1.0, 1.0) * 2.0 - corner
    idx = torch.floor(0.5 * n * (1.0 - corner)).clamp(0, n - 1).to(I64)
    at = idx.gather(1, chord(idx).argmin(1, keepdim=True))[:, 0]
    fm, f2 = fib[k - 1], fib[k + 2]
    off = torch.stack([torch.zeros_like(k), fm, -fm, f0, -f0, f1, -f1, f2, -f2], -1)
    twice = torch.zeros_like(off, dtype=torch.bool)
    twice[:, 1:3] = (fm == f0)[:, None]
    for _ in range(32):
        cand = at[:, None] + off
        ok = (cand >= 0) & (cand < n) & ~twice
        d = torch.where(ok, chord(cand.clamp(0, n - 1)), math.inf)
        best = cand.gather(1, d.argmin(1, keepdim=True))[:, 0]
        if bool((best == at).all()):
            break
        at = best
    d, order = torch.sort(d, dim=1, stable=True)
    return torch.where(torch.isinf(d), -1, cand.gather(1, order))[:, :K], d[:, :K]


def _exact_points(case, seed):
    s = prepare(case, seed)
    pts, q = _sf_points(case["n"]), s["query"].double()
    w = torch.empty((case["nq"], case["K"]), dtype=F64, device=DEV)
    for a in range(0, case["nq"], 1 << 19):
        part = q[a:a + (1 << 19)]
        _, d = _nearest(pts, part / part.norm(dim=1, keepdim=True), case["K"])
        w[a:a + (1 << 19)] = (1.0 - torch.sqrt(d) / math.sqrt(4.0 * math.pi / case["n"])).clamp_min(0.0)
    return pts, None, w


def _camera_rays(cam, W, H):
    eye = torch.tensor(np.float32(cam.eye), device=DEV, dtype=F64)
    fwd = torch.tensor(np.float32(cam.target), device=DEV, dtype=F64) - eye
    fwd = fwd / fwd.norm()
    right = torch.linalg.cross(fwd, torch.tensor(np.float32(cam.up), device=DEV, dtype=F64))
    right = right / right.norm()
    up = torch.linalg.cross(right, fwd)
    th = math.tan(0.5 * float(np.float32(cam.vfov)))
    x = (2.0 * (torch.arange(W, device=DEV, dtype=F64) + 0.5) / W - 1.0) * th * W / H
    y = (1.0 - 2.0 * (torch.arange(H, device=DEV, dtype=F64) + 0.5) / H) * th
    d = fwd + right * x[None, :, None] + up * y[:, None, None]
    return eye, (d / d.norm(dim=-1, keepdim=True)).reshape(-1, 3)


def _exact_lookup(case, seed):
    s = prepare(case, seed)
    M, N, K, W, H = case["M"], case["N"], case["K"], case["W"], case["H"]
    rows, lf = s["prm"].rows, s["lf"].view(-1, 3)
    rad = float(np.float32(R))
    po = _sf_points(M)
    pd = po if M == N else _sf_points(N)
    img = torch.zeros((case["views"], H * W, 3), dtype=F64, device=DEV)
    d_lf = torch.zeros((rows * N, 3), dtype=F64, device=DEV) if case["kind"] == "l2" else None
    step = 1 << 19
    for v, cam in enumerate(s["cams"]):
        eye, dirs = _camera_rays(cam, W, H)
        for a in range(0, H * W, step):
            d = dirs[a:a + step]
            b = d @ eye
            disc = b * b - (eye @ eye - rad * rad)
            hit = torch.nonzero(disc > 1e-6 * rad * rad)[:, 0]
            if not len(hit):
                continue
            d, b, sq = d[hit], b[hit], torch.sqrt(disc[hit])
            qo, qd = eye + d * (-b - sq)[:, None], eye + d * (-b + sq)[:, None]
            i, do = _nearest(po, qo / qo.norm(dim=1, keepdim=True), K)
            j, dd = _nearest(pd, qd / qd.norm(dim=1, keepdim=True), K)
            if K == 1:
                w = (i < rows).double()[:, :, None]
            else:
                wo = (1.0 - torch.sqrt(do) / math.sqrt(4.0 * math.pi / M)).clamp_min(0.0) * ((i >= 0) & (i < rows))
                wd = (1.0 - torch.sqrt(dd) / math.sqrt(4.0 * math.pi / N)).clamp_min(0.0) * (j >= 0)
                wo, wd = torch.nan_to_num(wo), torch.nan_to_num(wd)
                w = wo[:, :, None] * wd[:, None, :]
                if M == N:
                    w = w * (i[:, :, None] != j[:, None, :])
                tot = w.sum((1, 2), keepdim=True)
                w = torch.where(tot > 0.0, w / tot.clamp_min(1e-300), 0.0)
            t = (i.clamp(0, rows - 1)[:, :, None] * N + j.clamp_min(0)[:, None, :]).view(len(hit), -1)
            w = w.reshape(len(hit), -1)
            out = torch.zeros((len(hit), 3), dtype=F64, device=DEV)
            for p in range(t.shape[1]):
                out += w[:, p, None] * lf[t[:, p]].double()
            img[v, a + hit] = out
            if d_lf is not None:
                g = out - s["target"].view(case["views"], -1, 3)[v, a + hit].double()
                for p in range(t.shape[1]):
                    d_lf.index_add_(0, t[:, p], w[:, p, None] * g)
    img = img.view(case["views"], H, W, 3)
    if d_lf is not None:
        return img, d_lf.view(rows, N, 3)
    return (img, None) if case["nn"] else img


def _exact_metrics(case, seed):
    s = prepare(case, seed)
    a, b = (s[k].double().permute(0, 3, 1, 2) for k in ("a", "b"))
    H, W = case["H"], case["W"]
    g = torch.exp(-torch.arange(-5, 6, dtype=F64) ** 2 / 4.5)
    g = (g / g.sum()).tolist()

    def blur(x):
        x = sum(w * x[..., t:t + W - 10] for t, w in enumerate(g))
        return sum(w * x[..., t:t + H - 10, :] for t, w in enumerate(g))

    ma, mb = blur(a), blur(b)
    va, vb, cab = blur(a * a) - ma * ma, blur(b * b) - mb * mb, blur(a * b) - ma * mb
    c1, c2 = 0.01 ** 2, 0.03 ** 2
    ssim = ((2 * ma * mb + c1) * (2 * cab + c2) / ((ma * ma + mb * mb + c1) * (va + vb + c2))).mean((1, 2, 3))

    wx = 2.0 * math.pi * torch.fft.fftfreq(W, dtype=F64, device=DEV)[None, :]
    wy = 2.0 * math.pi * torch.fft.fftfreq(H, dtype=F64, device=DEV)[:, None]
    r, theta = torch.hypot(wx, wy), torch.atan2(wy.expand(H, W), wx.expand(H, W))
    sums = lambda x: (lambda y: sum(y[..., t:t + H - 6, :] for t in range(7)))(  # noqa: E731
        sum(x[..., t:t + W - 6] for t in range(7)))
    K, cw = 49 * 0.01 ** 2, torch.zeros(case["n"], dtype=F64, device=DEV)
    for m in range(case["n"]):
        fa, fb = torch.fft.fft2(a[m]), torch.fft.fft2(b[m])
        for sc in range(2):
            lr = torch.log2(r / (math.pi / 2 ** (sc + 1)))
            radial = torch.where(lr.abs() < 1.0, torch.cos(0.5 * math.pi * lr), 0.0)
            for k in range(4):
                d = theta - math.pi * k / 4
                d = d - 2.0 * math.pi * torch.round(d / (2.0 * math.pi))
                f = torch.nan_to_num(radial * torch.where(d.abs() < 0.5 * math.pi, torch.cos(d) ** 3, 0.0))
                ca, cb = torch.fft.ifft2(fa * f), torch.fft.ifft2(fb * f)
                cr = ca * cb.conj()
                num = 2.0 * torch.hypot(sums(cr.real), sums(cr.imag)) + K
                cw[m] += (num / (sums(ca.abs() ** 2) + sums(cb.abs() ** 2) + K)).mean() / 8
    return ssim, cw


def _philox(k, s, c2, blk, seed):
    """Philox4x32-10 block of counter (k, s, c2, blk) as four 64-bit integer tensors."""
    mask = 0xFFFFFFFF

    def mul(c, x):
        p0, p1 = c * (x & 0xFFFF), c * (x >> 16)
        return (p1 + (p0 >> 16)) >> 16, ((p1 << 16) + p0) & mask

    c0, c1, c3 = k, s, blk
    k0, k1 = seed & mask, seed >> 32
    for _ in range(10):
        ha, la = mul(0xD2511F53, c0)
        hb, lb = mul(0xCD9E8D57, c2)
        c0, c1, c2, c3 = hb ^ c1 ^ k0, lb, ha ^ c3 ^ k1, la
        k0, k1 = (k0 + 0x9E3779B9) & mask, (k1 + 0xBB67AE85) & mask
    return c0, c1, c2, c3


class _Tracer:
    """The volumetric path tracer, one tensor lane per sample."""

    def __init__(self, s):
        self.p, self.m, self.l = s["prm"], s["med"], s["light"]
        v = s["vol"]
        n = v.dims[0]
        self.n, self.vol = n, v.data.view(n, n, n)
        self.lut, self.scale = self.m.lut.double(), float(np.float32(self.m.scale))
        self.vmin, self.span = v.vmin, v.vmax - v.vmin
        self.G = max(1, self.p.grid)
        top = 1.25 * self.scale * self.lut[:, 3].max()
        self.maj = top.reshape(1, 1, 1) if self.p.grid == 0 else self._cells(top)
        self.maj = self.maj.float().double()

    def _cells(self, top):
        n, G, last = self.n, self.G, self.lut.shape[0] - 1
        out = torch.empty((G, G, G), dtype=F64, device=DEV)
        lo = [max((2 * c * n - G) // (2 * G) - 1, 0) for c in range(G)]
        hi = [min((2 * (c + 1) * n - G) // (2 * G) + 2, n - 1) for c in range(G)]
        e = torch.arange(last + 1, device=DEV)
        for z in range(G):
            for y in range(G):
                for x in range(G):
                    b = self.vol[lo[z]:hi[z] + 1, lo[y]:hi[y] + 1, lo[x]:hi[x] + 1]
                    u = ((torch.stack(b.aminmax()).double() - self.vmin) / self.span).clamp(0.0, 1.0) * last
                    u = u.floor().clamp_max(last - 1)
                    a = torch.where((e >= u[0]) & (e <= u[1] + 1), self.lut[:, 3], 0.0).max()
                    out[z, y, x] = torch.maximum(1.25 * self.scale * a, top / 256.0)
        return out

    def medium(self, x):
        n = self.n
        g = ((x + 1.0) * (n / 2.0) - 0.5).clamp(0.0, n - 1.0)
        i = g.floor().clamp_max(n - 2).to(I64)
        f = g - i
        at = (i[:, 2] * n + i[:, 1]) * n + i[:, 0]
        flat, c = self.vol.reshape(-1), 0.0
        for o in range(8):
            w = 1.0
            for a in range(3):
                w = w * (f[:, a] if o >> a & 1 else 1.0 - f[:, a])
            c = c + w * flat[at + (o & 1) + n * (o >> 1 & 1) + n * n * (o >> 2)].double()
        u = ((c - self.vmin) / self.span).clamp(0.0, 1.0) * (self.lut.shape[0] - 1)
        l0 = u.floor().clamp_max(self.lut.shape[0] - 2).to(I64)
        return torch.lerp(self.lut[l0], self.lut[l0 + 1], (u - l0)[:, None])

    @staticmethod
    def clip(x, d):
        inv = 1.0 / d
        a, b = (-1.0 - x) * inv, (1.0 - x) * inv
        tn = torch.minimum(a, b).amax(-1).clamp_min(0.0)
        tf = torch.maximum(a, b).amin(-1)
        return tn, tf, tn < tf

    def walk(self, x, d, t, tend, tau):
        """t where the variate tau is spent cell by cell, and the majorant there; t >= tend: left the segment."""
        G, w = self.G, 2.0 / self.G
        sb = torch.zeros_like(t)
        live = torch.nonzero(t < tend)[:, 0]
        t = t.clone()
        mid = x + d * t[:, None]
        cell = ((mid + 1.0) / w).floor().clamp(0, G - 1)
        while len(live):
            c, dl, xl = cell[live], d[live], x[live]
            plane = -1.0 + (c + (dl > 0)) * w
            tx = torch.where(dl == 0, math.inf, (plane - xl) / dl)
            exit_, axis = tx.min(-1)
            te = torch.minimum(exit_, tend[live])
            ci = c.to(I64).clamp(0, G - 1)
            m = self.maj[ci[:, 2], ci[:, 1], ci[:, 0]]
            room = m * (te - t[live]).clamp_min(0.0)
            here = tau[live] < room
            t[live] = torch.where(here, t[live] + tau[live] / m.clamp_min(1e-300), te)
            tau = tau.clone()
            tau[live] -= room
            sb[live] = m
            step = torch.zeros_like(c).scatter_(1, axis[:, None], torch.sign(dl.gather(1, axis[:, None])))
            cell[live] = c + step
            live = live[~here & (te < tend[live])]
        return t, sb

    def draw(self, k, s, b, purpose, pair):
        r = _philox(k, s, (b << 8 | purpose) + torch.zeros_like(k), pair >> 1, self.p.seed)
        odd = (pair & 1).bool()
        u = [torch.where(odd, r[2 + w], r[w]) for w in (0, 1)]
        return [(v >> 8).double() * 2.0 ** -24 for v in u]

    @staticmethod
    def turn(n, base, A, u):
        sg = torch.where(n[:, 2] >= 0, 1.0, -1.0).double()
        a = -1.0 / (sg + n[:, 2])
        b = n[:, 0] * n[:, 1] * a
        t1 = torch.stack([1.0 + sg * n[:, 0] ** 2 * a, sg * b, -sg * n[:, 0]], -1)
        t2 = torch.stack([b, sg + n[:, 1] ** 2 * a, -n[:, 1]], -1)
        ang = 2.0 * math.pi * u
        return base + t1 * (A * torch.cos(ang))[:, None] + t2 * (A * torch.sin(ang))[:, None]

    def radiance(self, k, s, x, d):
        """Radiance of samples s of rays k (64-bit integers) from x along d."""
        p, l, g = self.p, self.l, float(np.float32(self.p.g))
        vec = lambda v: torch.tensor(np.float32(v), device=DEV, dtype=F64)  # noqa: E731
        T, L = torch.ones_like(x), torch.zeros_like(x)
        lane = torch.arange(len(k), device=DEV)  # samples still on their way
        zero = torch.zeros_like(k)
        for b in range(p.max_bounces):
            tn, tf, hit = self.clip(x[lane], d[lane])
            L[lane[~hit]] += T[lane[~hit]] * vec(l.env)
            lane, t, tf = lane[hit], tn[hit], tf[hit]
            real, n = [], (1 if b == 0 else 0)
            colour = torch.zeros_like(T)
            while len(lane):
                u, v = self.draw(k[lane], s[lane], b, 1, zero[lane] + n)
                t, sb = self.walk(x[lane], d[lane], t, tf, -torch.log1p(-u))
                out = t >= tf
                L[lane[out]] += T[lane[out]] * vec(l.env)
                lane, t, tf, sb, v = (q[~out] for q in (lane, t, tf, sb, v))
                y = x[lane] + d[lane] * t[:, None]
                rgba = self.medium(y)
                take = v * sb < self.scale * rgba[:, 3]
                x[lane[take]] = y[take]
                colour[lane[take]] = rgba[take, :3].clamp(0.0, 1.0)
                real.append(lane[take])
                lane, t, tf = lane[~take], t[~take], tf[~take]
                n += 1
            lane = torch.cat(real).sort()[0] if real else lane
            T[lane] *= colour[lane]
            lane = lane[(T[lane] != 0).any(-1)]
            if not len(lane):
                break
            self.light_sample(k, s, x, d, T, L, lane, b, g, vec)
            if b == p.max_bounces - 1:
                break
            u0, u1 = self.draw(k[lane], s[lane], b, 2, zero[lane] + 1)
            if abs(g) < 1e-3:
                mu = 1.0 - 2.0 * u0
            else:
                q = (1.0 - g * g) / (1.0 - g + 2.0 * g * u0)
                mu = ((1.0 + g * g - q * q) / (2.0 * g)).clamp(-1.0, 1.0)
            d[lane] = self.turn(d[lane], d[lane] * mu[:, None], torch.sqrt((1.0 - mu * mu).clamp_min(0.0)), u1)
        return L

    def light_sample(self, k, s, x, d, T, L, lane, b, g, vec):
        l = self.l
        u0, u1 = self.draw(k[lane], s[lane], b, 2, torch.zeros_like(lane))
        if l.kind == 0:
            om = vec(l.dir)
            om = (om / om.norm()).expand(len(lane), 3)
            le, dist = vec(l.radiance).expand(len(lane), 3), torch.full((len(lane),), math.inf, dtype=F64, device=DEV)
        else:
            e1, e2 = vec(l.e1), vec(l.e2)
            v = vec(l.corner) + e1 * u0[:, None] + e2 * u1[:, None] - x[lane]
            dist = v.norm(dim=-1)
            om = v / dist[:, None]
            nrm = torch.linalg.cross(e1, e2)
            le = vec(l.radiance) * ((-(om @ nrm)).clamp_min(0.0) / dist ** 2)[:, None]
        mu = (d[lane] * om).sum(-1)
        C = T[lane] * le * ((1.0 - g * g) / (4.0 * math.pi) / (1.0 + g * g - 2.0 * g * mu) ** 1.5)[:, None]
        _, tf, hit = self.clip(x[lane], om)
        te = torch.where(hit, torch.minimum(tf, dist), 0.0)
        Tr, t = torch.ones_like(te), torch.zeros_like(te)
        live, n = torch.nonzero(te > 0)[:, 0], 2
        while len(live):
            u, _ = self.draw(k[lane[live]], s[lane[live]], b, 2, torch.zeros_like(live) + n)
            t[live], sb = self.walk(x[lane[live]], om[live], t[live], te[live], -torch.log1p(-u))
            inside = t[live] < te[live]
            live, sb = live[inside], sb[inside]
            sig = self.scale * self.medium(x[lane[live]] + om[live] * t[live, None])[:, 3]
            Tr[live] *= 1.0 - sig / sb
            n += 1
        L[lane] += C * Tr[:, None]


def _exact_trace(case, seed):
    s = prepare(case, seed)
    tr, p = _Tracer(s), s["prm"]
    if case["kind"] == "render":
        W, H = case["W"], case["H"]
        rays = [_camera_rays(c, W, H) for c in s["cams"]]
        d = torch.cat([r[1] for r in rays])
        x = torch.cat([r[0].expand(H * W, 3) for r in rays])
        keep, n = torch.arange(len(d), device=DEV), None
    else:
        po, pd = _sf_points(p.M), _sf_points(p.N)
        i = torch.arange(p.rows, device=DEV).repeat_interleave(p.N)
        j = torch.arange(p.N, device=DEV).repeat(p.rows)
        keep = torch.nonzero(i != j)[:, 0] if p.M == p.N else torch.arange(len(i), device=DEV)
        n = po[i[keep]]
        d = pd[j[keep]] - n
        d = d / d.norm(dim=-1, keepdim=True)
        x = n * float(np.float32(R))
    out = torch.zeros((case["views"] * H * W if n is None else p.rows * p.N, 3), dtype=F64, device=DEV)
    for smp in range(p.spp):
        sv = torch.full_like(keep, smp)
        x0 = x.clone()
        if n is not None:
            u0, u1 = tr.draw(keep, sv, 0, 1, torch.zeros_like(keep))
            x0 = tr.turn(n, x, 2.0 * float(np.float32(R)) / math.sqrt(p.M) * torch.sqrt(u0), u1)
        out[keep] += tr.radiance(keep, sv, x0, d.clone())
    out /= p.spp
    return out.view((case["views"], case["H"], case["W"], 3) if n is None else (p.rows, p.N, 3))


def exact(case, seed):
    kind = case["kind"]
    if kind == "points":
        return _exact_points(case, seed)
    if kind in ("lookup", "l2"):
        return _exact_lookup(case, seed)
    if kind == "metrics":
        return _exact_metrics(case, seed)
    if kind in ("generate", "render") and not case.get("surface", False):
        # (fields of over two million samples take too long; the step's and
        # the training's gradients come of such fields)
        px = case["views"] * case["W"] * case["H"] if kind == "render" else (case["rows"] or case["M"]) * case["N"]
        if px * case["spp"] <= 2000000:
            return _exact_trace(case, seed)
    return None
