"""What this package is timed on: the calls its users make, over the range of sizes they make them at.

A user renders with the package.  Offline, they march rays through a density
cloud or a fire, stochastically or with every tap as the reference image.  In
real time they look up 2-D textures for each pixel: magnified, minified on a
plane with isotropic or anisotropic footprints, compressed, mapped from three
planes.  For learned assets they train a latent lattice, then decode it in 2-D
or march it in 3-D.  ``listed`` has one case for each of these at the size
that ``bench.py`` or the tests use, some at ragged sizes; ``draw`` gives more
over the range of each.

``exact`` evaluates the same call in float64 with torch alone.  The integer
decisions (which texel a sample reads, at which level) follow the binary32
contract of ``include/sf.h``, since they define the estimate; all values are
float64.
"""
import math

import numpy as np
import torch

import paper_2407_06107_amd as sf
from paper_2407_06107_amd import inputs

SIDE = 0.25  # world side of every volume
FILTERS = {"linear": sf.SF_LINEAR, "bspline": sf.SF_BSPLINE3, "keys": sf.SF_KEYS3, "ewa": sf.SF_EWA}
MODES = {"before": sf.SF_BEFORE, "after": sf.SF_AFTER_EXACT, "stochastic": sf.SF_STOCHASTIC, "split": sf.SF_SPLIT}
SHADES = {"none": sf.SF_SHADE_NONE, "ggx": sf.SF_SHADE_GGX, "normal": sf.SF_SHADE_GGX_NORMAL}
TAPS = {"linear": 2, "bspline": 4, "keys": 4}


# --------------------------------------------------------------------- cases
def listed():
    return [
        # the offline renderer's inner loop: one voxel per step of a million rays through a 512^3 cloud
        dict(name="march_cloud", kind="march", nx=512, ny=512, nz=512, half=True, brick=3, filter="bspline",
             mode="stochastic", pixels=256, rays=16, steps=256, spp=1),
        # the reference image of the same view: all 64 taps of every step, shaded before they are summed
        dict(name="march_reference", kind="march", nx=512, ny=512, nz=512, half=True, brick=3, filter="bspline",
             mode="after", pixels=256, rays=16, steps=256, spp=1),
        # a fire seen by black-body emission, a ragged grid
        dict(name="emission_fire", kind="emission", nx=420, ny=372, nz=333, half=True, brick=3, filter="bspline",
             mode="stochastic", pixels=201, rays=16, steps=200, spp=1, footprint=0.0),
        # a small magnified texture, 16 samples a query: the smallest call, where launching it counts
        dict(name="texture_magnified", kind="texture", width=64, height=64, eight=False, levels=1, wrap="repeat",
             image="noise", view="uniform", n=4096, filter="bspline", mode="stochastic", spp=16, shade="ggx"),
        # a frame of a textured plane, one sample a pixel: the real-time path
        dict(name="texture_plane", kind="texture", width=4096, height=4096, eight=True, levels=13, wrap="repeat",
             image="waves", view="plane", n=1920 * 1080, filter="bspline", mode="stochastic", spp=1, shade="ggx"),
        # the reference image of that frame: 16 taps on two levels, each shaded
        dict(name="texture_reference", kind="texture", width=4096, height=4096, eight=True, levels=13, wrap="repeat",
             image="waves", view="plane", n=1920 * 1080, filter="bspline", mode="after", spp=1, shade="ggx"),
        # a minified checkerboard under elliptical footprints, one texel a pixel, a ragged frame
        dict(name="footprint_ewa", kind="footprint", width=4096, height=4096, levels=13, image="checker",
             pixels_x=1279, pixels_y=719, filter="ewa", mode="stochastic", aniso=16, spp=1, shade="ggx"),
        # a compressed texture mapped on a sphere from three planes, one plane and one texel a pixel
        dict(name="triplanar_dct", kind="triplanar", width=4096, height=4096, dct=True, pixels_x=1920, pixels_y=1080,
             filter="linear", mode="stochastic", pick_plane=True, spp=1),
        # compressing that texture with all its levels
        dict(name="dct_encode", kind="encode", width=4096, height=4096),
        # a neural texture, one decode a query
        dict(name="neural_texture", kind="neural_texture", res_x=1024, res_y=1024, fp8=False, n=2097152,
             filter="bspline", mode="stochastic", spp=1, shade="ggx"),
        # a neural density volume, one decode a step
        dict(name="neural_volume", kind="neural_volume", nx=256, ny=256, nz=256, fp8=True, filter="bspline",
             pixels=256, rays=16, steps=128, spp=1),
        # fitting that volume: one optimiser step on a batch of lattice points
        dict(name="neural_training", kind="training", res_x=256, res_y=256, res_z=256, channels=16, batch=262144,
             fp32=False),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["march", "march", "emission", "texture", "texture", "texture", "footprint", "footprint",
                       "triplanar", "encode", "neural_texture", "neural_volume", "training"])
    if kind in ("march", "emission"):
        c = dict(kind=kind, half=rng.random() < 0.75, brick=rng.choice([0, 2, 3, 3]))
        for a in ("nx", "ny", "nz"):
            c[a] = _log_int(rng, 40, 512)
        c.update(filter=rng.choice(["linear", "bspline", "bspline"]),
                 mode=rng.choice(["stochastic", "stochastic", "before", "after"]), rays=rng.choice([1, 16, 16]),
                 steps=_log_int(rng, 20, 256), pixels=_log_int(rng, 24, 256), spp=1)
        if c["mode"] != "stochastic" and not (c["half"] and c["brick"] and kind == "march"):
            c["pixels"] = min(c["pixels"], 128)     # dearer a step than the listed reference image
        if kind == "emission":
            c["footprint"] = rng.choice([0.0, 0.5]) if c["mode"] == "stochastic" else 0.0
        if c["mode"] == "stochastic" and c["rays"] == 1:
            c["spp"] = rng.choice([1, 4, 16])
        return c
    if kind == "texture":
        c = dict(kind=kind, eight=rng.random() < 0.7, wrap=rng.choice(["repeat", "repeat", "clamp"]))
        top = 4096 if c["eight"] else 1024
        c["width"], c["height"] = _log_int(rng, 48, top), _log_int(rng, 48, top)
        c["levels"] = rng.choice([1, _full(c), _full(c)])
        c["view"] = rng.choice(["uniform", "plane", "plane"])
        c["n"] = _log_int(rng, 1000, 1920 * 1080)
        c["mode"] = rng.choice(["stochastic", "stochastic", "before", "after", "split"])
        c["filter"] = rng.choice(["linear", "bspline", "bspline", "keys"])
        c["spp"] = rng.choice([1, 1, 4, 16]) if c["mode"] in ("stochastic", "split") else 1
        c["shade"] = rng.choice(["ggx", "ggx", "normal", "none"])
        c["image"] = "normals" if c["shade"] == "normal" else rng.choice(["waves", "noise"])
        return c
    if kind == "footprint":
        c = dict(kind=kind, width=_log_int(rng, 512, 4096))
        c["height"] = max(256, min(4096, int(c["width"] * rng.choice([1, 1, 0.5, 0.77]))))
        c["levels"] = _full(c)
        c["pixels_x"], c["pixels_y"] = _log_int(rng, 64, 1920), _log_int(rng, 64, 1080)
        c["filter"] = rng.choice(["ewa", "ewa", "linear", "bspline"])
        c["mode"] = rng.choice(["stochastic", "stochastic", "before", "after"])
        c["aniso"] = rng.choice([4, 16]) if c["filter"] == "ewa" else rng.choice([16, 64])
        c["spp"] = rng.choice([1, 1, 4]) if c["mode"] == "stochastic" else 1
        c["shade"] = rng.choice(["ggx", "normal"])
        c["image"] = "normals" if c["shade"] == "normal" else "checker"
        return c
    if kind == "triplanar":
        return dict(kind=kind, width=_log_int(rng, 128, 4096), height=_log_int(rng, 128, 4096),
                    dct=rng.random() < 0.6, pixels_x=_log_int(rng, 64, 1920), pixels_y=_log_int(rng, 64, 1080),
                    filter=rng.choice(["linear", "bspline"]), mode=rng.choice(["stochastic", "stochastic", "before"]),
                    pick_plane=rng.random() < 0.7, spp=1)
    if kind == "encode":
        return dict(kind=kind, width=_log_int(rng, 64, 4096), height=_log_int(rng, 64, 4096))
    if kind == "neural_texture":
        c = dict(kind=kind, res_x=_log_int(rng, 64, 1024), res_y=_log_int(rng, 64, 1024), fp8=rng.random() < 0.3,
                 n=_log_int(rng, 1000, 2097152), filter=rng.choice(["linear", "bspline", "bspline"]),
                 mode=rng.choice(["stochastic", "stochastic", "before", "after"]), shade=rng.choice(["ggx", "none"]))
        c["spp"] = rng.choice([1, 1, 4]) if c["mode"] == "stochastic" else 1
        return c
    if kind == "neural_volume":
        return dict(kind=kind, nx=_log_int(rng, 32, 256), ny=_log_int(rng, 32, 256), nz=_log_int(rng, 32, 256),
                    fp8=rng.random() < 0.7, filter=rng.choice(["linear", "bspline"]), pixels=_log_int(rng, 16, 256),
                    rays=rng.choice([1, 16, 16]), steps=_log_int(rng, 16, 160), spp=1)
    if rng.random() < 0.4:
        c = dict(kind="training", res_x=_log_int(rng, 128, 1024), res_y=_log_int(rng, 128, 1024), res_z=1, channels=8)
    else:
        c = dict(kind="training", res_x=_log_int(rng, 48, 256), res_y=_log_int(rng, 48, 256),
                 res_z=_log_int(rng, 48, 256), channels=16)
    c["batch"] = _log_int(rng, 1000, min(262144, c["res_x"] * c["res_y"] * c["res_z"]))
    c["fp32"] = rng.random() < 0.25
    return c


def _full(c):
    return int(math.floor(math.log2(max(c["width"], c["height"])))) + 1


# -------------------------------------------------------------------- inputs
def _gen(seed, salt, device="cuda"):
    return torch.Generator(device=device).manual_seed(int(seed) * 16 + salt)


def _waves(w, h, seed, salt, gradient=False):
    """A tileable band-limited field in [-1, 1] (or its two slopes), waves of amplitude 1/frequency."""
    g = np.random.default_rng([int(seed), salt])
    x = torch.arange(w, device="cuda", dtype=torch.float32) * (2 * math.pi / w)
    y = torch.arange(h, device="cuda", dtype=torch.float32) * (2 * math.pi / h)
    outs = [torch.zeros(h, w, device="cuda") for _ in range(2 if gradient else 1)]
    total = 0.0
    for _ in range(24):
        mag, ang, phase = math.exp(g.random() * math.log(min(w, h) / 2)), g.random() * 2 * math.pi, g.random() * 2 * math.pi
        fx, fy = round(mag * math.cos(ang)), round(mag * math.sin(ang))
        amp = 1.0 / max(1.0, math.hypot(fx, fy))
        a = (fx * x)[None, :] + (fy * y + phase)[:, None]
        if gradient:
            outs[0] += amp * fx * torch.cos(a)
            outs[1] += amp * fy * torch.cos(a)
            total += amp * math.hypot(fx, fy)
        else:
            outs[0] += amp * torch.sin(a)
            total += amp
    return [o / total for o in outs]


def _image(kind, w, h, seed):
    """[h, w, 4] float32 on the GPU: albedo (or an encoded normal) and roughness."""
    if kind == "noise":
        img = torch.rand(h, w, 4, device="cuda", generator=_gen(seed, 1))
        img[..., 3] = 0.05 + 0.95 * img[..., 3]
        return img
    if kind == "waves":
        return torch.stack([0.5 + 0.5 * _waves(w, h, seed, c)[0] for c in range(4)], -1)
    if kind == "checker":
        g = np.random.default_rng(int(seed))
        cx, cy = max(2, w // 64), max(2, h // 64)
        ox, oy = int(g.integers(cx)), int(g.integers(cy))
        light = (((torch.arange(w, device="cuda") + ox) // cx)[None, :]
                 + ((torch.arange(h, device="cuda") + oy) // cy)[:, None]) & 1
        lo, hi = torch.tensor([0.04, 0.04, 0.04, 0.1], device="cuda"), torch.tensor([0.9, 0.9, 0.9, 0.9], device="cuda")
        return torch.where(light[..., None] > 0, hi, lo)
    gx, gy = _waves(w, h, seed, 7, gradient=True)
    n = torch.stack([-3.0 * gx, -3.0 * gy, torch.ones_like(gx)], -1)
    n = n / n.norm(dim=-1, keepdim=True)
    return torch.cat([0.5 * (n + 1.0), torch.full_like(gx, 0.15)[..., None]], -1)


def _pyramid(c, seed, image, eight, levels):
    """Level arrays as a program holds them (uint8 or float32 on the host)."""
    x = _image(image, c["width"], c["height"], seed).permute(2, 0, 1)[None]
    out = []
    for l in range(levels):
        if l:
            x = torch.nn.functional.adaptive_avg_pool2d(x, (max(1, c["height"] >> l), max(1, c["width"] >> l)))
        lv = x[0].permute(1, 2, 0).contiguous()
        out.append(((lv.clamp(0, 1) * 255).round().to(torch.uint8) if eight else lv).cpu().numpy())
    return out


def _tex(c, seed, image, eight, levels, wrap="repeat"):
    lv = _pyramid(c, seed, image, eight, levels)
    return lv, dict(wrap=sf.SF_WRAP_REPEAT if wrap == "repeat" else sf.SF_WRAP_CLAMP,
                    mip=sf.SF_MIP_LINEAR if levels > 1 else sf.SF_MIP_NONE)


def _frame(n):
    """A 16:9 frame of about n pixels, cut to n."""
    w = max(1, int(round(math.sqrt(n * 16 / 9))))
    return w, -(-n // w)


def _queries(c, seed):
    g = np.random.default_rng([int(seed), 3])
    if c["view"] == "uniform":
        q = np.empty((c["n"], 3), np.float32)
        q[:, :2] = g.random((c["n"], 2))
        q[:, 2] = g.random(c["n"]) * (c["levels"] - 1)
        return torch.from_numpy(q).cuda()
    w, h = _frame(c["n"])
    q = inputs.plane_queries(w, h, tex_size=max(c["width"], c["height"]), levels=c["levels"])[:c["n"]]
    q[:, :2] += g.random(2).astype(np.float32)
    return torch.from_numpy(q).cuda()


def _cloud(c, seed):
    grid = inputs.cloud_grid(max(c["nx"], c["ny"], c["nz"]), seed=int(seed) % 100003, device="cuda")
    return grid[:c["nz"], :c["ny"], :c["nx"]].contiguous()


def _rays(c, seed):
    r = inputs.ortho_rays(c["pixels"], c["rays"], side=SIDE, seed=int(seed) + 1, strata=4 if c["rays"] == 16 else 0)
    return torch.from_numpy(r).cuda()


def _smp(c, seed):
    return sf.sampling(FILTERS[c["filter"]], MODES[c.get("mode", "stochastic")], c["spp"], seed=_hash_seed(seed))


def _hash_seed(seed):
    return (int(seed) * 2654435761 + 12345) & 0xFFFFFFFF


def _mlp(cin, cout, seed):
    """Packed FP32 parameters of the size a fitted network has (He-normal, small biases)."""
    g = _gen(seed, 5)
    parts = []
    for a, b in ((cin, 64), (64, 64), (64, cout)):
        parts += [torch.randn(a * b, device="cuda", generator=g) * math.sqrt(2.0 / a),
                  torch.randn(b, device="cuda", generator=g) * 0.1]
    if cout == 4:      # outputs around 1/2: albedo and roughness
        parts[4] *= 0.15
        parts[5] += 0.5
    return torch.cat(parts)


def _latents(npts, ch, seed):
    return torch.randn(npts * ch, device="cuda", generator=_gen(seed, 6)) * 0.5


def _grid2(c, seed):
    lat = _latents(c["res_x"] * c["res_y"], 8, seed)
    return sf.sf_neural_quantize(lat, 2, (c["res_x"], c["res_y"]), 8,
                                 sf.SF_LATENT_FP8E4M3 if c["fp8"] else sf.SF_LATENT_BF16)


def _grid3(c, seed):
    lat = _latents(c["nx"] * c["ny"] * c["nz"], 16, seed)
    return sf.sf_neural_quantize(lat, 3, (c["nx"], c["ny"], c["nz"]), 16,
                                 sf.SF_LATENT_FP8E4M3 if c["fp8"] else sf.SF_LATENT_BF16, 3, (0.0, 0.0, 0.0),
                                 (c["nx"] / SIDE, c["ny"] / SIDE, c["nz"] / SIDE))


def _volume_mlp(seed):
    p = _mlp(16, 1, seed)
    p[16 * 64 + 64 + 64 * 64 + 64:] *= 10.0   # the density scale, folded into the last layer
    return p


def _training(c, seed):
    """State after 100 steps: latents, their moments at the size of their gradients, targets in [0, 1]."""
    npts, ch, out = c["res_x"] * c["res_y"] * c["res_z"], c["channels"], 4 if c["channels"] == 8 else 1
    g = _gen(seed, 8)
    par = _mlp(ch, out, seed)
    scale = 1.0 / c["batch"]
    rn = lambda k, s: torch.randn(k, device="cuda", generator=g) * s  # noqa: E731
    return dict(latents=_latents(npts, ch, seed), params=par, m_lat=rn(npts * ch, 0.1 * scale),
                v_lat=rn(npts * ch, scale).square_().add_(scale * scale), m_par=rn(par.numel(), 1e-3),
                v_par=rn(par.numel(), 1e-2).square_().add_(1e-4),
                targets=torch.rand(npts, out, device="cuda", generator=g),
                batch=torch.randperm(npts, device="cuda", generator=g)[:c["batch"]].to(torch.int32))


LR_LATENT, LR_MLP, STEP = 1e-2, 1e-3, 101


def prepare(case, seed):
    c, kind = case, case["kind"]
    s = dict(case=c, smp=None if kind in ("encode", "training") else _smp(c, seed), ggx=sf.ggx())
    if kind in ("march", "emission"):
        data = _cloud(c, seed)
        if kind == "emission":
            data = inputs.temperature_grid(data)
        if not c["half"]:
            data = data.float()
        s["vol"] = sf.Volume(data, side=SIDE, brick_log2=c["brick"] or None)
        s["rays"] = _rays(c, seed)
        if kind == "emission":
            s["footprint"] = c["footprint"] * inputs.ortho_pixel_width(c["pixels"], SIDE)
    elif kind == "texture":
        lv, how = _tex(c, seed, c["image"], c["eight"], c["levels"], c["wrap"])
        s["tex"], s["q"] = sf.Texture2D(lv, **how), _queries(c, seed)
    elif kind == "footprint":
        lv, how = _tex(c, seed, c["image"], True, c["levels"])
        s["tex"], s["q"] = sf.Texture2D(lv, **how), _footprints(c, seed)
    elif kind == "triplanar":
        lv, how = _tex(c, seed, "waves", True, _full(c))
        s["tex"] = sf.Texture2D(lv, **how)
        if c["dct"]:
            s["tex"] = sf.Texture2D.dct(s["tex"])
        s["q"] = _sphere(c, seed)
    elif kind == "encode":
        lv, how = _tex(c, seed, "waves", True, _full(c))
        s["tex"] = sf.Texture2D(lv, **how)
    elif kind == "neural_texture":
        s["grid"], s["mlp"] = _grid2(c, seed), sf.MLP(_mlp(8, 4, seed), 8, 4)
        s["q"] = torch.from_numpy(inputs.queries_uniform(c["n"], seed=int(seed))).cuda()
    elif kind == "neural_volume":
        s["grid"], s["mlp"], s["rays"] = _grid3(c, seed), sf.MLP(_volume_mlp(seed), 16, 1), _rays(c, seed)
    else:
        t = _training(c, seed)
        st = sf.TrainState(t["latents"], t["params"], c["channels"], 4 if c["channels"] == 8 else 1,
                           compute=sf.SF_TRAIN_FP32 if c["fp32"] else sf.SF_TRAIN_BF16)
        for a, b in ((st.m_lat, "m_lat"), (st.v_lat, "v_lat"), (st.m_par, "m_par"), (st.v_par, "v_par")):
            a.copy_(t[b])
        s.update(state=st, batch=t["batch"], targets=t["targets"])
    return s


def _footprints(c, seed):
    q = inputs.plane_queries_aniso(c["pixels_x"], c["pixels_y"])
    q[:, :2] += np.random.default_rng([int(seed), 3]).random(2).astype(np.float32)
    return torch.from_numpy(q).cuda()


def _sphere(c, seed):
    q = inputs.sphere_queries(c["pixels_x"], c["pixels_y"], tex_size=max(c["width"], c["height"]), levels=_full(c))
    return torch.from_numpy(q).cuda()


def run(state):
    c, s = state["case"], state
    kind = c["kind"]
    if kind == "march":
        return sf.sf_raymarch(s["vol"], s["rays"], c["steps"], s["smp"])
    if kind == "emission":
        return sf.sf_raymarch_emission(s["vol"], s["rays"], c["steps"], s["smp"], footprint=s["footprint"])
    if kind == "texture":
        return sf.sf_filter2d(s["tex"], s["q"], s["smp"], SHADES[c["shade"]], s["ggx"])
    if kind == "footprint":
        return sf.sf_filter2d_aniso(s["tex"], s["q"], s["smp"], c["aniso"], SHADES[c["shade"]], s["ggx"])
    if kind == "triplanar":
        return sf.sf_triplanar(s["tex"], s["q"], s["smp"], 1.0, 1 if c["pick_plane"] else 0, sf.SF_SHADE_GGX, s["ggx"])
    if kind == "encode":
        t = sf.Texture2D.dct(s["tex"])
        return [t.buffer, t.ranges]
    if kind == "neural_texture":
        return sf.sf_neural_decode(s["grid"], s["mlp"], s["q"], s["smp"], SHADES[c["shade"]], s["ggx"])
    if kind == "neural_volume":
        return sf.sf_neural_raymarch(s["grid"], s["mlp"], s["rays"], c["steps"], s["smp"])
    st = s["state"]
    loss = sf.sf_neural_train_step(st, s["batch"], s["targets"], LR_LATENT, LR_MLP, step=STEP)
    return [loss, st.params, st.m_par, st.v_par, st.latents, st.m_lat, st.v_lat]


# ------------------------------------------------------------------ the work
def work(case):
    """Inputs read once, outputs written once, and the arithmetic of the estimate."""
    c, kind = case, case["kind"]
    if kind in ("march", "emission"):
        n, esz = c["pixels"] ** 2 * c["rays"], 2 if c["half"] else 4
        steps = n * c["steps"] * c["spp"]
        taps = 1 if c["mode"] == "stochastic" else TAPS[c["filter"]] ** 3
        per_tap = {"stochastic": 4, "before": 2, "after": 12}[c["mode"]]
        out = 3 if kind == "emission" else 1
        return dict(bytes=n * (32 + 4 * out) + min(c["nx"] * c["ny"] * c["nz"], steps * taps) * esz,
                    flops=steps * (60 + taps * per_tap * out))
    if kind in ("texture", "footprint", "triplanar"):
        tap1 = 1 if c["mode"] == "stochastic" else (30 if c["filter"] == "ewa" else TAPS[c["filter"]] ** 2)
        if kind == "texture":
            n, esz, rec, lv = c["n"], 4 if c["eight"] else 16, 12, 2 if c["levels"] > 1 else 1
        else:
            n, esz, lv = c["pixels_x"] * c["pixels_y"], 4, 2
            rec = 24 if kind == "footprint" else 32
            if kind == "triplanar":
                n = int(0.41 * n)                     # the pixels that see the sphere
                esz = 0.25 if c["dct"] else 4
        lookups = n * c["spp"] * tap1 * (1 if c["mode"] in ("stochastic", "split") else lv)
        out = 16 if c.get("shade") == "none" else 12
        texels = c["width"] * c["height"] * (4 / 3 if lv > 1 else 1)
        return dict(bytes=n * (rec + out) + min(texels * esz, lookups * esz), flops=lookups * 40 + n * c["spp"] * 40)
    if kind == "encode":
        px = c["width"] * c["height"] * 4 / 3
        return dict(bytes=px * 4.25, flops=px * 4 * 2 * (3 + 6 / 8))
    if kind == "neural_texture":
        dec = c["n"] * c["spp"] * (1 if c["mode"] == "stochastic" else TAPS[c["filter"]] ** 2)
        esz = 8 if c["fp8"] else 16
        return dict(bytes=c["n"] * 24 + min(c["res_x"] * c["res_y"], dec) * esz, flops=dec * 9728)
    if kind == "neural_volume":
        n = c["pixels"] ** 2 * c["rays"]
        dec = n * c["steps"] * c["spp"]
        return dict(bytes=n * 36 + min(c["nx"] * c["ny"] * c["nz"], dec) * (16 if c["fp8"] else 32), flops=dec * 10368)
    ch, out = c["channels"], 4 if c["channels"] == 8 else 1
    return dict(bytes=c["batch"] * (4 + 4 * out + 6 * 4 * ch), flops=c["batch"] * 6 * (ch * 64 + 64 * 64 + 64 * out))


# ------------------------------------------------- the same calls in float64
def _d(x):
    return x.double() if isinstance(x, torch.Tensor) else float(np.float32(x))


def _fma(a, b, c):
    """Binary32 fused multiply-add: the product is exact in float64."""
    return (_d(a) * _d(b) + _d(c)).float()


def _f(x):
    return float(np.float32(x))


def _div(a, b):
    """Binary32 quotient a / b by a number (torch multiplies by a number's reciprocal instead)."""
    return a / torch.full_like(a, b)


def _pcg4d(x, y, z, w):
    M = 0xFFFFFFFF
    v = [(k * 1664525 + 1013904223) & M for k in (x, y, z, w)]
    for last in (False, True):
        v[0] = (v[0] + v[1] * v[3]) & M
        v[1] = (v[1] + v[2] * v[0]) & M
        v[2] = (v[2] + v[0] * v[1]) & M
        v[3] = (v[3] + v[1] * v[2]) & M
        if not last:
            v = [k ^ (k >> 16) for k in v]
    return v


def _key(q, s, k, seed):
    t = lambda v: torch.tensor(v, device="cuda", dtype=torch.int64)  # noqa: E731
    return [(v >> 8).float() * 2.0 ** -24 for v in _pcg4d(q, t(s), t(k), t(_hash_seed(seed)))]


def _pick(filt, t, u):
    """Tap offset of the uniform u: binary32 running sums, ties advance."""
    if filt == "linear":
        return (u >= 1.0 - t).long()
    s, t2 = 1.0 - t, t * t
    c0 = ((s * s) * s) * _f(1 / 6)
    c1 = c0 + _fma(-t2, _fma(-0.5, t, 1.0), _f(2 / 3))
    c2 = 1.0 - (t2 * t) * _f(1 / 6)
    return -1 + (u >= c0).long() + (u >= c1).long() + (u >= c2).long()


def _weights(filt, t):
    """(first tap offset, float64 weights)."""
    t = t.double()
    s = 1.0 - t
    if filt == "linear":
        return 0, [s, t]
    if filt == "bspline":
        return -1, [s ** 3 / 6, 2 / 3 - t * t * (1 - t / 2), 2 / 3 - s * s * (1 - s / 2), t ** 3 / 6]
    return -1, [-t * s * s / 2, 1 + t * t * (1.5 * t - 2.5), 1 + s * s * (1.5 * s - 2.5), -s * t * t / 2]


def _dirs():
    unit = lambda v: np.array(v, np.float64) / np.linalg.norm(v)  # noqa: E731
    r32 = lambda v: v.astype(np.float32).astype(np.float64)  # noqa: E731
    wo, wi = r32(unit((0.2, 0.3, 1.0))), r32(unit((-0.4, 0.1, 1.0)))
    h = wo + wi
    return wo, wi, h / np.linalg.norm(h)


def _shade(kind, c):
    """Texel values [..., 4] to radiance [..., 3] (or themselves): GGX + Lambert times the cosine."""
    if kind == "none":
        return c
    wo, wi, h = _dirs()
    f0, bias, scale = _f(0.04), _f(0.05), _f(0.95)
    F = f0 + (1 - f0) * (1 - float(wi @ h)) ** 5
    a2 = (bias + scale * c[..., 3]) ** 4
    if kind == "ggx":
        no, ni, nh = wo[2], wi[2], h[2]
        d = nh * nh * (a2 - 1) + 1
        g = lambda x: 2 / (x + torch.sqrt(a2 + (1 - a2) * x * x))  # noqa: E731
        spec = a2 / (math.pi * d * d) * g(no) * g(ni) * F / 4
        return ni * (c[..., :3] / math.pi + spec[..., None])
    m = 2 * c[..., :3] - 1
    ln = m.norm(dim=-1, keepdim=True)
    m = torch.where(ln > 0, m / ln, torch.tensor([0.0, 0.0, 1.0], device="cuda", dtype=torch.float64))
    dot = lambda v: m @ torch.tensor(v, device="cuda")  # noqa: E731
    no, ni, nh = dot(wo).clamp(min=0), dot(wi).clamp(min=0), dot(h)
    cross = torch.linalg.cross(m, torch.tensor(h, device="cuda").expand_as(m))
    d = (cross * cross).sum(-1) + nh * nh * a2
    g = lambda x: 2 / (x + torch.sqrt(a2 + (1 - a2) * x * x))  # noqa: E731
    spec = a2 / (math.pi * d * d) * g(no) * g(ni) * F / 4
    return (ni * (0.5 / math.pi + spec))[..., None].expand(*spec.shape, 3)


class _Levels:
    """The texels of all levels as one float64 lookup."""

    def __init__(self, levels, wrap):
        self.eight, self.wrap = levels[0].dtype == np.uint8, wrap
        self.flat = torch.cat([torch.from_numpy(lv.reshape(-1, 4)) for lv in levels]).cuda()
        size = [lv.shape[0] * lv.shape[1] for lv in levels]
        t = lambda v: torch.tensor(v, device="cuda", dtype=torch.int64)  # noqa: E731
        self.off, self.n = t(np.concatenate([[0], np.cumsum(size)[:-1]]).tolist()), len(levels)
        self.w, self.h = t([lv.shape[1] for lv in levels]), t([lv.shape[0] for lv in levels])

    def texel(self, l, x, y):
        w, h = self.w[l], self.h[l]
        if self.wrap == "repeat":
            x, y = torch.remainder(x, w), torch.remainder(y, h)
        else:
            x, y = torch.minimum(x.clamp(min=0), w - 1), torch.minimum(y.clamp(min=0), h - 1)
        return self.fetch(l, x, y, w)

    def fetch(self, l, x, y, w):
        v = self.flat[self.off[l] + y * w + x]
        return v.double() / 255.0 if self.eight else v.double()

    def coord(self, u):
        return u - torch.floor(u) if self.wrap == "repeat" else u.clamp(0.0, 1.0)

    def raster(self, u, v, l):
        px, py = _fma(u, self.w[l].float(), -0.5), _fma(v, self.h[l].float(), -0.5)
        fx, fy = torch.floor(px), torch.floor(py)
        return fx.long(), fy.long(), px - fx, py - fy

    def pair(self, lam):
        """Levels floor and floor + 1 of lambda and the fraction."""
        if self.n == 1:
            z = torch.zeros_like(lam, dtype=torch.int64)
            return z, z, torch.zeros_like(lam)
        lc = lam.clamp(0.0, float(self.n - 1))
        fl = torch.floor(lc)
        return fl.long(), (fl.long() + 1).clamp(max=self.n - 1), lc - fl

    def recon(self, filt, u, v, l, shade="none"):
        """Sum over the taps of w * shade(texel) on level l."""
        ix, iy, tx, ty = self.raster(u, v, l)
        first, wx = _weights(filt, tx)
        _, wy = _weights(filt, ty)
        tot = 0.0
        for b in range(len(wy)):
            for a in range(len(wx)):
                tot = tot + (wx[a] * wy[b])[:, None] * _shade(shade, self.texel(l, ix + first + a, iy + first + b))
        return tot

    def blend(self, filt, u, v, lam, shade="none"):
        l0, l1, f = self.pair(lam)
        r = self.recon(filt, u, v, l0, shade)
        if self.n > 1:
            f = f.double()[:, None]
            r = (1 - f) * r + f * self.recon(filt, u, v, l1, shade)
        return r


class _Blocks(_Levels):
    """The same over DCT blocks: a texel is decoded from its block's six coefficients a channel."""

    def __init__(self, tex, wrap):
        d, self.wrap, self.n = tex.desc, wrap, tex.desc.levels
        t = lambda v: torch.tensor(v, device="cuda", dtype=torch.int64)  # noqa: E731
        self.words = (tex.buffer[:tex.buffer.numel() // 16 * 16].view(torch.int32).long() & 0xFFFFFFFF).view(-1, 4)
        self.off = t([tex.offsets[l] // 16 for l in range(self.n)])
        self.w = t([max(1, d.width >> l) for l in range(self.n)])
        self.h = t([max(1, d.height >> l) for l in range(self.n)])
        self.range = tex.ranges.double().view(-1, 4)
        k, x = torch.arange(3, dtype=torch.float64)[:, None], torch.arange(8, dtype=torch.float64)[None, :]
        b = torch.cos((2 * x + 1) * k * math.pi / 16) / 2
        b[0] = math.sqrt(1 / 8)
        self.basis = b.cuda()

    def fetch(self, l, x, y, w):
        wd = self.words[self.off[l] + (y >> 3) * ((w + 7) >> 3) + (x >> 3)]
        R, bx, by = self.range[l], self.basis[:, x & 7], self.basis[:, y & 7]
        v = (wd & 127).double() * (8 / 127) * (bx[0] * by[0])[:, None]
        for k, (p, q) in enumerate(((1, 0), (0, 1), (0, 2), (1, 1), (2, 0))):
            v = v + (((wd >> (7 + 5 * k)) & 31) - 15).double() * R / 15 * (bx[p] * by[q])[:, None]
        return v.clamp(0.0, 1.0)


def _mean(total, spp):
    return total / spp


def _keys_estimate(lv, l, ix, iy, tx, ty, q, s, seed, shade):
    """Positivised Keys: one tap of the positive, one of the negative product weights."""
    def axis(t):
        r = 1.0 - t
        m0, m3 = (0.5 * t) * (r * r), (0.5 * r) * (t * t)
        p1 = _fma(t * t, _fma(1.5, t, -2.5), 1.0)
        p2 = _fma(r * r, _fma(1.5, r, -2.5), 1.0)
        return m0, m0 + m3, p1, p1 + p2
    (m0x, Mx, p1x, Px), (m0y, My, p1y, Py) = axis(tx), axis(ty)
    w, w2 = _key(q, s, 0, seed), _key(q, s, 1, seed)
    A, B, C, D = Px * Py, Mx * My, Px * My, Mx * Py
    pos = lambda u, P, p1: torch.where(u * P < p1, 0, 1)  # noqa: E731
    neg = lambda u, M, m0: torch.where(u * M < m0, -1, 2)  # noqa: E731
    a, b = w[2] * (A + B) < A, w2[2] * (C + D) < C
    ox = torch.where(a, pos(w[0], Px, p1x), neg(w[0], Mx, m0x))
    oy = torch.where(a, pos(w[1], Py, p1y), neg(w[1], My, m0y))
    nx = torch.where(b, pos(w2[0], Px, p1x), neg(w2[0], Mx, m0x))
    ny = torch.where(b, neg(w2[1], My, m0y), pos(w2[1], Py, p1y))
    wx, wy = _weights("keys", tx)[1], _weights("keys", ty)[1]
    P = (wx[1] + wx[2]) * (wy[1] + wy[2]) + (wx[0] + wx[3]) * (wy[0] + wy[3])
    N = -(wx[1] + wx[2]) * (wy[0] + wy[3]) - (wx[0] + wx[3]) * (wy[1] + wy[2])
    has = ((C + D) > 0)[:, None]
    vp, vn = _shade(shade, lv.texel(l, ix + ox, iy + oy)), _shade(shade, lv.texel(l, ix + nx, iy + ny))
    return P[:, None] * vp - torch.where(has, N[:, None] * vn, torch.zeros_like(vn))


def _exact_texture(c, seed):
    lv = _Levels(_pyramid(c, seed, c["image"], c["eight"], c["levels"]), c["wrap"])
    q = _queries(c, seed)
    u, v, lam = lv.coord(q[:, 0]), lv.coord(q[:, 1]), q[:, 2]
    if c["mode"] == "before":
        return _shade(c["shade"], lv.blend(c["filter"], u, v, lam))
    if c["mode"] == "after":
        return lv.blend(c["filter"], u, v, lam, c["shade"])
    l0, l1, f = lv.pair(lam)
    i = torch.arange(q.shape[0], device="cuda")
    tot = 0.0
    for s in range(c["spp"]):
        w = _key(i, s, 0, seed)
        l = torch.where(w[3] >= 1.0 - f, l1, l0)
        if c["mode"] == "split":
            tot = tot + _shade(c["shade"], lv.recon(c["filter"], u, v, l))
            continue
        ix, iy, tx, ty = lv.raster(u, v, l)
        if c["filter"] == "keys":
            tot = tot + _keys_estimate(lv, l, ix, iy, tx, ty, i, s, seed, c["shade"])
        else:
            t = lv.texel(l, ix + _pick(c["filter"], tx, w[0]), iy + _pick(c["filter"], ty, w[1]))
            tot = tot + _shade(c["shade"], t)
    return _mean(tot, c["spp"])


# ln, log2, exp and cos/sin of the decision contract: fixed binary32 sequences
LN2_HI, LN2_LO = float.fromhex("0x1.62e4p-1"), _f(1.42860677e-6)


def _atanh_series(x):
    m, e = torch.frexp(x)
    low = m < _f(0.70710678)
    m, e = torch.where(low, m * 2.0, m), torch.where(low, e - 1, e).float()
    s = (m - 1.0) / (m + 1.0)
    z = s * s
    p = _fma(z, _f(1 / 9), _f(1 / 7))
    for k in (1 / 5, 1 / 3, 1.0):
        p = _fma(z, p, _f(k))
    return (2.0 * s) * p, e


def _log2c(x):
    ok = x >= 2.0 ** -126
    r, e = _atanh_series(torch.where(ok, x, torch.ones_like(x)))
    return torch.where(ok, _fma(r, _f(1.44269504), e), torch.full_like(x, -math.inf))


def _lnc(x):
    r, e = _atanh_series(x)
    return _fma(e, LN2_HI, _fma(e, LN2_LO, r))


def _expc(x):
    n = torch.floor(_fma(x, _f(1.44269504), 0.5))
    r = _fma(-n, LN2_LO, _fma(-n, LN2_HI, x))
    p = _fma(r, _f(1 / 5040), _f(1 / 720))
    for k in (1 / 120, 1 / 24, 1 / 6, 0.5, 1.0, 1.0):
        p = _fma(r, p, _f(k))
    return torch.where(x >= -80.0, torch.ldexp(p, n.clamp(min=-126)), torch.zeros_like(x))


def _sincos2pi(v):
    a = 4.0 * v
    qf = torch.floor(a)
    f, q = a - qf, qf.long() & 3
    fold = f > 0.5
    x = torch.where(fold, 1.0 - f, f) * _f(1.57079637)
    z = x * x
    sp = _fma(z, _f(1 / 362880), _f(-1 / 5040))
    for k in (1 / 120, -1 / 6, 1.0):
        sp = _fma(z, sp, _f(k))
    cp = _fma(z, _f(-1 / 3628800), _f(1 / 40320))
    for k in (-1 / 720, 1 / 24, -0.5, 1.0):
        cp = _fma(z, cp, _f(k))
    sn = x * sp
    c0, s0 = torch.where(fold, sn, cp), torch.where(fold, cp, sn)
    pick = lambda w: torch.where(q == 0, w[0], torch.where(q == 1, w[1], torch.where(q == 2, w[2], w[3])))  # noqa: E731
    return pick((c0, -s0, -c0, s0)), pick((s0, c0, -s0, -c0))


def _exact_footprint(c, seed):
    lv = _Levels(_pyramid(c, seed, c["image"], True, c["levels"]), "repeat")
    q = _footprints(c, seed)
    return _exact_ewa(c, seed, lv, q) if c["filter"] == "ewa" else _exact_aniso(c, seed, lv, q)


def _exact_aniso(c, seed, lv, q):
    W, H, A = float(c["width"]), float(c["height"]), float(c["aniso"])
    ax, ay, bx, by = W * q[:, 2], H * q[:, 3], W * q[:, 4], H * q[:, 5]
    la, lb = ax * ax + ay * ay, bx * bx + by * by
    swap = la > lb
    lmin, lmax = torch.sqrt(torch.where(swap, lb, la)), torch.sqrt(torch.where(swap, la, lb))
    lmin = torch.where(lmin * A < lmax, lmin * (lmax / (lmin * A)), lmin)
    lam = _log2c(lmin)
    if c["mode"] == "stochastic":
        i = torch.arange(q.shape[0], device="cuda")
        tot = 0.0
        for s in range(c["spp"]):
            w0, w1 = _key(i, s, 0, seed), _key(i, s, 1, seed)
            jx, jy = w0[0] - 0.5, w0[1] - 0.5
            u = lv.coord(_fma(jy, q[:, 4], _fma(jx, q[:, 2], q[:, 0])))
            v = lv.coord(_fma(jy, q[:, 5], _fma(jx, q[:, 3], q[:, 1])))
            l = torch.floor((lam + (w0[2] - 0.5)).clamp(0.0, float(lv.n - 1)) + 0.5).long()
            ix, iy, tx, ty = lv.raster(u, v, l)
            t = lv.texel(l, ix + _pick(c["filter"], tx, w1[0]), iy + _pick(c["filter"], ty, w1[1]))
            tot = tot + _shade(c["shade"], t)
        return _mean(tot, c["spp"])
    probes = torch.ceil(lmax / lmin).clamp(1.0, A)
    mu, mv = torch.where(swap, q[:, 2], q[:, 4]), torch.where(swap, q[:, 3], q[:, 5])
    after = c["mode"] == "after"
    tot = 0.0
    for k in range(int(probes.max())):
        o = (k + 0.5) / probes - 0.5
        u, v = lv.coord(_fma(o, mu, q[:, 0])), lv.coord(_fma(o, mv, q[:, 1]))
        r = lv.blend(c["filter"], u, v, lam, c["shade"] if after else "none")
        tot = tot + torch.where((k < probes)[:, None], r / probes.double()[:, None], torch.zeros_like(r))
    return tot if after else _shade(c["shade"], tot)


def _exact_ewa(c, seed, lv, q):
    W, H, A = float(c["width"]), float(c["height"]), float(c["aniso"])
    jsx, jtx, jsy, jty = W * q[:, 2], H * q[:, 3], W * q[:, 4], H * q[:, 5]
    vss, vtt, vst = jsx * jsx + jsy * jsy, jtx * jtx + jty * jty, jsx * jtx + jsy * jty
    dj = jsx * jty - jtx * jsy
    det = dj * dj
    half, mean = (vss - vtt) * 0.5, (vss + vtt) * 0.5
    lp = mean + torch.sqrt(half * half + vst * vst)
    s1 = torch.sqrt(lp)
    minor = dj.abs() / s1
    lim = minor * A < s1
    lm, mlim = det / lp, _div(s1, A)
    k = torch.where(lp > lm, (mlim * mlim - lm) / (lp - lm), torch.ones_like(lp))
    vss, vtt = torch.where(lim, vss + k * (lp - vss), vss), torch.where(lim, vtt + k * (lp - vtt), vtt)
    vst, det = torch.where(lim, vst - k * vst, vst), torch.where(lim, lp * (mlim * mlim), det)
    lod = _log2c(torch.where(lim, mlim, minor)).clamp(min=0.0)
    wide = lod > float(lv.n - 1)
    last = torch.full_like(lod, lv.n - 1, dtype=torch.int64)
    zero = torch.zeros_like(last)
    u, v = lv.coord(q[:, 0]), lv.coord(q[:, 1])
    fl = torch.floor(lod)
    frac = lod - fl
    e2 = _expc(torch.tensor([-2.0], device="cuda"))

    def level(l):
        wl, hl = lv.w[l].float(), lv.h[l].float()
        fs, ft = _div(wl, W), _div(hl, H)
        lss, ltt, lst = vss * (fs * fs), vtt * (ft * ft), vst * (fs * ft)
        a, b = lss + 1.0, ltt + 1.0
        D = ((det * ((fs * fs) * (ft * ft)) + lss) + ltt) + 1.0
        s, t = u * wl - 0.5, v * hl - 0.5
        ex, ey = torch.sqrt(a), torch.sqrt(b)
        box = [torch.ceil(s - ex), torch.floor(s + ex), torch.ceil(t - ey), torch.floor(t + ey)]
        return (s, t, b / D, a / D, -(2.0 * lst) / D, *[x.long() for x in box])

    def cells(lev):
        """Cells of the boxes in scan order: (x, y, binary32 weight)."""
        s, t, qss, qtt, q2, x0, x1, y0, y1 = lev
        for y in range(int((y1 - y0).max()) + 1):
            for x in range(int((x1 - x0).max()) + 1):
                ix, iy = x0 + x, y0 + y
                ds, dt = ix.float() - s, iy.float() - t
                r2 = (qss * (ds * ds) + qtt * (dt * dt)) + q2 * (ds * dt)
                w = torch.where((r2 < 1.0) & (ix <= x1) & (iy <= y1), _expc(-2.0 * r2) - e2, torch.zeros_like(r2))
                yield ix, iy, torch.where(w > 0.0, w, torch.zeros_like(w))

    if c["mode"] == "stochastic":
        i = torch.arange(q.shape[0], device="cuda")
        tot = 0.0
        for smp in range(c["spp"]):
            w = _key(i, smp, 0, seed)
            l = (fl.clamp(0, lv.n - 1).long() + (w[3] >= 1.0 - frac).long()).clamp(max=lv.n - 1)
            lev = level(l)
            S = torch.zeros_like(lod)
            for _, _, wt in cells(lev):
                S = S + wt
            thr, S = w[0] * S, torch.zeros_like(lod)
            px, py, done = zero, zero, torch.zeros_like(wide)
            for x, y, wt in cells(lev):
                take = (wt > 0.0) & ~done
                S, px, py = torch.where(take, S + wt, S), torch.where(take, x, px), torch.where(take, y, py)
                done = done | (take & (S > thr))
            t = lv.texel(torch.where(wide, last, l), torch.where(wide, zero, px), torch.where(wide, zero, py))
            tot = tot + _shade(c["shade"], t)
        return _mean(tot, c["spp"])
    after, tot = c["mode"] == "after", 0.0
    for k, p in ((0, 1.0 - frac.double()), (1, frac.double())):
        l = (fl.clamp(0, lv.n - 1).long() + k).clamp(max=lv.n - 1)
        num, den = 0.0, 0.0
        for x, y, wt in cells(level(l)):
            wt = wt.double()
            num = num + wt[:, None] * _shade(c["shade"] if after else "none", lv.texel(l, x, y))
            den = den + wt
        tot = tot + (p / den)[:, None] * num
    one = lv.texel(last, zero, zero)
    tot = torch.where(wide[:, None], _shade(c["shade"], one) if after else one, tot)
    return tot if after else _shade(c["shade"], tot)


def _exact_triplanar(c, seed):
    if c["dct"]:
        lv = _Blocks(prepare(c, seed)["tex"], "repeat")
    else:
        lv = _Levels(_pyramid(c, seed, "waves", True, _full(c)), "repeat")
    q = _sphere(c, seed)
    p, lam = q[:, :3], q[:, 6]
    w = (q[:, 3:6] * q[:, 3:6]).square()
    Wf = (w[:, 0] + w[:, 1]) + w[:, 2]
    b = q[:, 3:6].double() ** 4
    b = b / b.sum(1, keepdim=True)
    uv = [(p[:, 1], p[:, 2]), (p[:, 0], p[:, 2]), (p[:, 0], p[:, 1])]
    i = torch.arange(q.shape[0], device="cuda")
    h = _key(i, 0, 0, seed)
    plane = (h[2] >= w[:, 0] / Wf).long() + (h[2] >= (w[:, 0] + w[:, 1]) / Wf).long()
    l0, l1, f = lv.pair(lam)
    l = torch.where(h[3] >= 1.0 - f, l1, l0)

    def one(u, v):
        u, v = lv.coord(u), lv.coord(v)
        if c["mode"] != "stochastic":
            return lv.blend(c["filter"], u, v, lam)
        ix, iy, tx, ty = lv.raster(u, v, l)
        return _shade("ggx", lv.texel(l, ix + _pick(c["filter"], tx, h[0]), iy + _pick(c["filter"], ty, h[1])))

    if c["pick_plane"]:
        r = one(torch.where(plane == 0, uv[0][0], uv[1][0]), torch.where(plane == 2, uv[2][1], uv[0][1]))
    else:
        r = sum(b[:, j:j + 1] * one(*uv[j]) for j in range(3))
    return r if c["mode"] == "stochastic" else _shade("ggx", r)


def _geometry(rays, scale, steps):
    """Binary32 entry point, step and step length of each ray, and which rays march."""
    t0, t1 = rays[:, 6], rays[:, 7]
    dt = _div(t1 - t0, float(steps))
    E, G = [], []
    for a in range(3):
        A = _fma(rays[:, a] - 0.0, _f(scale[a]), -0.5)
        B = rays[:, 3 + a] * _f(scale[a])
        E.append(_fma(t0, B, A))
        G.append(dt * B)
    return E, G, dt, t1 > t0


def _planck(T):
    """Spectral radiance at the three wavelengths, [..., 3]; nothing at or below 0 K."""
    h, cl, k = 6.62607015e-34, 299792458.0, 1.380649e-23
    out = []
    for nm in (700.0, 546.1, 435.8):
        lam = nm * 1e-9
        x = h * cl / (lam * k) / T.clamp(min=1e-30)
        out.append(torch.where(T > 0, 2 * h * cl * cl / lam ** 5 / torch.expm1(x) * 1e-9, torch.zeros_like(T)))
    return torch.stack(out, -1)


def _exact_volume(c, seed):
    fire = c["kind"] == "emission"
    data = _cloud(c, seed)
    if fire:
        data = inputs.temperature_grid(data)
    n3 = (c["nx"], c["ny"], c["nz"])
    scale = [a / SIDE for a in n3]
    flat, rays = data.reshape(-1), _rays(c, seed)
    E, G, dt, hit = _geometry(rays, scale, c["steps"])
    i = torch.arange(rays.shape[0], device="cuda")
    dtd = dt.double()

    def voxel(x, y, z):
        ok = (x >= 0) & (x < n3[0]) & (y >= 0) & (y < n3[1]) & (z >= 0) & (z < n3[2])
        return torch.where(ok, flat[torch.where(ok, (z * n3[1] + y) * n3[0] + x, 0)].double(), 0.0)

    foot = c.get("footprint", 0.0) * inputs.ortho_pixel_width(c["pixels"], SIDE)
    if foot > 0.0:
        dx, dy, dz = rays[:, 3], rays[:, 4], rays[:, 5]
        sg = torch.copysign(torch.ones_like(dz), dz)
        a = -1.0 / (sg + dz)
        b = (dx * dy) * a
        e1, e2 = (1.0 + ((sg * dx) * dx) * a, sg * b, -sg * dx), (b, sg + (dy * dy) * a, -dy)
        FA, FB = ([(_f(foot) * e[k]) * _f(scale[k]) for k in range(3)] for e in (e1, e2))
    mean = 0.0
    for s in range(c["spp"]):
        tot = torch.ones_like(dtd) if c["mode"] == "after" and not fire else 0.0
        for k in range(c["steps"]):
            p = [_fma(k + 0.5, G[a], E[a]) for a in range(3)]
            if foot > 0.0:
                w = _key(i, s | 0x80000000, k, seed)
                r = torch.sqrt(-2.0 * _lnc(1.0 - w[0]))
                cs, sn = _sincos2pi(w[1])
                g1, g2 = r * cs, r * sn
                p = [_fma(g2, FB[a], _fma(g1, FA[a], p[a])) for a in range(3)]
            i0 = [torch.floor(x) for x in p]
            t = [x - f for x, f in zip(p, i0)]
            i0 = [f.long() for f in i0]
            if c["mode"] == "stochastic":
                w = _key(i, s, k, seed)
                v = voxel(*[i0[a] + _pick(c["filter"], t[a], w[a]) for a in range(3)])
                tot = tot + (_planck(v) if fire else v)
                continue
            first, wx = _weights(c["filter"], t[0])
            wy, wz = _weights(c["filter"], t[1])[1], _weights(c["filter"], t[2])[1]
            acc = 0.0
            for cz in range(len(wz)):
                for by in range(len(wy)):
                    wyz = wy[by] * wz[cz]
                    for ax in range(len(wx)):
                        v = voxel(i0[0] + first + ax, i0[1] + first + by, i0[2] + first + cz)
                        wt = wx[ax] * wyz
                        if c["mode"] == "before":
                            acc = acc + wt * v
                        elif fire:
                            acc = acc + wt[:, None] * _planck(v)
                        else:
                            acc = acc + wt * torch.exp(-dtd * v)
            if fire:
                tot = tot + (_planck(acc) if c["mode"] == "before" else acc)
            elif c["mode"] == "before":
                tot = tot + acc
            else:
                tot = tot * acc
        mean = mean + (tot * dtd[:, None] if fire else tot if c["mode"] == "after" else torch.exp(-dtd * tot))
        if c["mode"] != "stochastic":
            break
    mean = _mean(mean, c["spp"] if c["mode"] == "stochastic" else 1)
    return torch.where(hit[:, None], mean, 0.0) if fire else torch.where(hit, mean, 1.0)


def _dct_ranges(c, seed):
    """Largest |AC| of the kept coefficients a level and channel."""
    k, x = torch.arange(3, dtype=torch.float64)[:, None], torch.arange(8, dtype=torch.float64)[None, :]
    b = torch.cos((2 * x + 1) * k * math.pi / 16) / 2
    b[0] = math.sqrt(1 / 8)
    b = b.cuda()
    out = []
    for lv in _pyramid(c, seed, "waves", True, _full(c)):
        v = torch.from_numpy(lv).cuda()
        h, w = v.shape[:2]
        yy = torch.arange(-(-h // 8) * 8, device="cuda").clamp(max=h - 1)
        xx = torch.arange(-(-w // 8) * 8, device="cuda").clamp(max=w - 1)
        v = v[yy][:, xx].double().div_(255.0).view(yy.numel() // 8, 8, xx.numel() // 8, 8, 4)
        top = None
        for p, q in ((1, 0), (0, 1), (0, 2), (1, 1), (2, 0)):
            wgt = b[q][:, None, None, None] * b[p][None, None, :, None]
            m = (v * wgt[None]).sum((1, 3)).abs().amax((0, 1))
            top = m if top is None else torch.maximum(top, m)
        out.append(top)
    return torch.cat(out)


def _bf16_mlp(params, cin, cout):
    """The packed parameters rounded to bfloat16, as float64 matrices."""
    p, out, o = params.bfloat16().double(), [], 0
    for a, b in ((cin, 64), (64, 64), (64, cout)):
        out.append((p[o:o + a * b].view(a, b), p[o + a * b:o + a * b + b]))
        o += a * b + b
    return out


def _forward(mlp, z):
    (w1, b1), (w2, b2), (w3, b3) = mlp
    return torch.relu(torch.relu(z @ w1 + b1) @ w2 + b2) @ w3 + b3


def _operands(grid, idx, xyz):
    """Latents of lattice points as the decoder reads them: bfloat16 (E4M3 codes times their block's scale)."""
    d = grid.desc
    if d.format == sf.SF_LATENT_BF16:
        return grid.latents.view(torch.bfloat16).view(-1, d.channels)[idx].double()
    code = grid.latents.view(torch.float8_e4m3fn).view(-1, d.channels)[idx].float()
    nb = [-(-d.res[a] // (1 << d.block_log2)) for a in range(3)]
    bx, by, bz = (v >> d.block_log2 for v in xyz)
    return (code * grid.scales[(bz * nb[1] + by) * nb[0] + bx][:, None]).bfloat16().double()


def _exact_neural_texture(c, seed):
    grid, mlp = _grid2(c, seed), _bf16_mlp(_mlp(8, 4, seed), 8, 4)
    q = torch.from_numpy(inputs.queries_uniform(c["n"], seed=int(seed))).cuda()
    R = (c["res_x"], c["res_y"])
    p = [_fma(q[:, a] - torch.floor(q[:, a]), float(R[a]), -0.5) for a in range(2)]
    i0 = [torch.floor(x) for x in p]
    t = [x - f for x, f in zip(p, i0)]
    i0 = [f.long() for f in i0]

    def texel(x, y):
        x, y = torch.remainder(x, R[0]), torch.remainder(y, R[1])
        return _forward(mlp, _operands(grid, y * R[0] + x, (x, y, torch.zeros_like(x)))).clamp(0.0, 1.0)

    tot = 0.0
    if c["mode"] == "stochastic":
        i = torch.arange(c["n"], device="cuda")
        for s in range(c["spp"]):
            w = _key(i, s, 0, seed)
            tot = tot + _shade(c["shade"], texel(*[i0[a] + _pick(c["filter"], t[a], w[a]) for a in range(2)]))
        return _mean(tot, c["spp"])
    first, wx = _weights(c["filter"], t[0])
    wy = _weights(c["filter"], t[1])[1]
    for b in range(len(wy)):
        for a in range(len(wx)):
            v = texel(i0[0] + first + a, i0[1] + first + b)
            tot = tot + (wx[a] * wy[b])[:, None] * (_shade(c["shade"], v) if c["mode"] == "after" else v)
    return tot if c["mode"] == "after" else _shade(c["shade"], tot)


def _exact_neural_volume(c, seed):
    grid, mlp, rays = _grid3(c, seed), _bf16_mlp(_volume_mlp(seed), 16, 1), _rays(c, seed)
    n3 = (c["nx"], c["ny"], c["nz"])
    E, G, dt, hit = _geometry(rays, [a / SIDE for a in n3], c["steps"])
    i = torch.arange(rays.shape[0], device="cuda")
    tau = torch.zeros(rays.shape[0], device="cuda", dtype=torch.float64)
    for k in range(c["steps"]):
        p = [_fma(k + 0.5, G[a], E[a]) for a in range(3)]
        w = _key(i, 0, k, seed)
        x = []
        for a in range(3):
            f = torch.floor(p[a])
            x.append(f.long() + _pick(c["filter"], p[a] - f, w[a]))
        ok = hit.clone()
        for a in range(3):
            ok &= (x[a] >= 0) & (x[a] < n3[a])
        x = [torch.where(ok, v, 0) for v in x]
        y = _forward(mlp, _operands(grid, (x[2] * n3[1] + x[1]) * n3[0] + x[0], x))[:, 0]
        tau += torch.where(ok, y.clamp(min=0.0), 0.0)
    return torch.where(hit, torch.exp(-dt.double() * tau), 1.0)


def _exact_training(c, seed):
    t = _training(c, seed)
    ch, out = c["channels"], 4 if c["channels"] == 8 else 1
    idx = t["batch"].long()
    lat = t["latents"].view(-1, ch)
    leaves = [lat[idx].double().requires_grad_(True), t["params"].double().requires_grad_(True)]
    p, o, mats = leaves[1], 0, []
    for a, b in ((ch, 64), (64, 64), (64, out)):
        mats.append((p[o:o + a * b].view(a, b), p[o + a * b:o + a * b + b]))
        o += a * b + b
    loss = (_forward(mats, leaves[0]) - t["targets"][idx].double()).square().sum() / c["batch"]
    gz, gp = torch.autograd.grad(loss, leaves)
    c1, c2 = 1 - 0.9 ** STEP, 1 - 0.999 ** STEP

    def adam(x, m, v, g, lr):
        m, v = 0.9 * m.double() + 0.1 * g, 0.999 * v.double() + 0.001 * g * g
        return x.double() - lr * (m / c1) / (torch.sqrt(v / c2) + 1e-8), m, v

    np_, nm, nv = adam(t["params"], t["m_par"], t["v_par"], gp, LR_MLP)
    ml, vl = t["m_lat"].view(-1, ch), t["v_lat"].view(-1, ch)
    z, m, v = adam(lat[idx], ml[idx], vl[idx], gz, LR_LATENT)
    whole = []
    for base, rows in ((lat, z), (ml, m), (vl, v)):
        full = base.double()
        full[idx] = rows
        whole.append(full.reshape(-1))
    return [loss.detach().reshape(1), np_, nm, nv, *whole]


def exact(case, seed):
    kind = case["kind"]
    if kind in ("march", "emission"):
        return _exact_volume(case, seed)
    if kind == "texture":
        return _exact_texture(case, seed)
    if kind == "footprint":
        return _exact_footprint(case, seed)
    if kind == "triplanar":
        return _exact_triplanar(case, seed)
    if kind == "encode":
        return [None, _dct_ranges(case, seed)]   # the blocks are whole numbers
    if kind == "neural_texture":
        return _exact_neural_texture(case, seed)
    if kind == "neural_volume":
        return _exact_neural_volume(case, seed)
    return _exact_training(case, seed)
