"""The work this framework is measured on: calls a user's program makes, over the sizes it makes them at.

Every case is seeded synthetic lunar terrain (octaves of smooth noise plus bowl craters, as in
the library's own benchmark) with a sun a few degrees above the horizon.  The sun's azimuth comes
from the seed, its elevation from the case.  Sizes, spacings, ray caps and run schedules are the
benchmark's and the tests': 256^2 up to the 16384^2 polar tile, ragged shapes between.

``exact`` evaluates the same definitions in float64 with plain torch.  The descents commit to the
smallest of several bounds; where two of them are nearly equal either choice is a valid
evaluation, so a few rays differ from float64 by more than rounding.
"""
from __future__ import annotations

import math
import random

import torch
import torch.nn.functional as F

import paper_2005_06671_amd as ss

R_MOON = 1737400.0
DISC = math.radians(0.267)          # angular radius of the sun disc
DEV = "cuda"
LIMIT_RAYS = 150_000_000            # float64 reference: at most this many rays (about 20 s)

MODES = {"descent": ss.SS_MODE_DP, "uniform": ss.SS_MODE_UNIFORM, "exact": ss.SS_MODE_EXACT,
         "point": ss.SS_MODE_POINT}
RUNS = {"geometric": dict(),
        "555": dict(schedule=ss.SS_SCHED_EQUAL, n_prime0=5, n_segments=3),
        "5553": dict(schedule=ss.SS_SCHED_LIST, n_segments=4, n_prime_list=(5, 5, 5, 3))}


def listed():
    return [
        # the smallest call: one sun over a 256^2 tile, the mipmap built by the call
        dict(name="small 256", kind="cast", w=256, h=256, texel=20.0, amp=2000.0, craters=0,
             mode="descent", runs="geometric", elev=1.5, cap=0.0),
        # an ordinary tile cut to odd sides, whose spacing fits no power of two
        dict(name="ragged 1531 x 1019", kind="cast", w=1531, h=1019, texel=12.5, amp=2000.0,
             craters=60, mode="descent", runs="geometric", elev=1.1, cap=30000.0),
        # the flagship: a day's suns over a 4096^2 tile, replayed from a plan
        dict(name="plan 4096 x 8 suns", kind="plan", w=4096, h=4096, texel=5.0, amp=2000.0,
             craters=120, mode="descent", suns=8, cap=30000.0),
        # the largest: a polar tile at grazing sun, 60 km rays
        dict(name="polar 16384", kind="cast", w=16384, h=16384, texel=2.0, amp=4000.0,
             craters=200, mode="descent", runs="geometric", elev=0.2, cap=60000.0),
        # uneven tiles of a mosaic with a few suns, called once (no plan)
        dict(name="batched uneven", kind="batched", w=2048, h=1024, texel=10.0, amp=2000.0,
             craters=60, mode="descent", suns=6, cap=30000.0, tiles=4),
        # inverse rendering: forward and backward to the heights and the sun
        dict(name="train 2048", kind="train", w=2048, h=2048, texel=10.0, amp=2000.0, craters=120,
             mode="descent", elev=1.5, cap=30000.0, record=False),
        # the global minimum (branch and bound), with its pyramid built by the call
        dict(name="exact 2048", kind="cast", w=2048, h=2048, texel=10.0, amp=2000.0, craters=120,
             mode="exact", runs="geometric", elev=1.5, cap=30000.0),
        # the baseline everybody compares with: one-texel steps
        dict(name="uniform 1024", kind="cast", w=1024, h=1024, texel=20.0, amp=2000.0, craters=60,
             mode="uniform", runs="geometric", elev=1.5, cap=30000.0),
        # a rendered frame: view rays, then the paper's {5,5,5} shadow rays at the hits
        dict(name="frame 1920 x 1080", kind="frame", w=2048, h=2048, texel=10.0, amp=2000.0,
             craters=120, mode="point", runs="555", elev=1.5, cap=0.0, px=1920, py=1080),
        # gradients through the shadows of a small image's visible points
        dict(name="image train 512 x 384", kind="image_train", w=1024, h=1024, texel=10.0,
             amp=2000.0, craters=60, mode="descent", elev=2.0, cap=30000.0, px=512, py=384),
        # a working tile stitched from two cube-face sub-tiles across their seam
        dict(name="stitch 4096", kind="stitch", w=4096, h=4096, texel=5.0, amp=2000.0),
        # new terrain arrives: both pyramids over it
        dict(name="terrain 4096", kind="terrain", w=4096, h=4096, texel=5.0, amp=2000.0,
             craters=120),
    ]


def _side(rng, lo, hi):
    n = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    return max(lo, min(hi, n if rng.random() < 0.6 else (n + 8) // 16 * 16))


def draw(rng: random.Random):
    kind = rng.choice(["cast", "cast", "cast", "cast", "plan", "batched", "train", "train",
                       "frame", "image_train", "stitch", "terrain"])
    c = dict(kind=kind, amp=float(rng.choice([1000.0, 2000.0, 4000.0])),
             texel=float(rng.choice([2.0, 5.0, 7.5, 10.0, 12.5, 20.0])))
    elev = round(math.exp(rng.uniform(math.log(0.2), math.log(4.0))), 3)
    cap = float(rng.choice([0.0, 10000.0, 30000.0, 60000.0]))
    if kind == "cast":
        mode = rng.choice(["descent", "descent", "descent", "exact", "uniform", "point"])
        hi = {"descent": 6144, "point": 4096, "exact": 2048, "uniform": 1024}[mode]
        c.update(w=_side(rng, 96, hi), h=_side(rng, 96, hi), craters=40, mode=mode, elev=elev,
                 cap=cap, plane=rng.random() < 0.2,
                 runs=rng.choice(["geometric", "geometric", "555", "5553"])
                 if mode in ("descent", "point") else "geometric",
                 core=rng.random() < 0.25)
    elif kind in ("plan", "batched"):
        c.update(w=_side(rng, 128, 2048), h=_side(rng, 128, 2048), craters=40, cap=cap,
                 mode=rng.choice(["descent", "descent", "exact"]), suns=rng.randint(2, 8),
                 tiles=1 if kind == "plan" else rng.randint(2, 4))
    elif kind == "train":
        c.update(w=_side(rng, 128, 4096), h=_side(rng, 128, 4096), craters=40, elev=elev, cap=cap,
                 mode=rng.choice(["descent", "descent", "point"]), record=rng.random() < 0.3)
    elif kind in ("frame", "image_train"):
        c.update(w=_side(rng, 512, 2048), h=_side(rng, 512, 2048), craters=40, elev=elev,
                 texel=10.0, px=_side(rng, 160, 1920), py=_side(rng, 120, 1080))
        if kind == "frame":
            c.update(mode=rng.choice(["point", "descent"]), runs=rng.choice(["555", "5553"]),
                     cap=0.0)
        else:
            c.update(mode="descent", cap=cap)
    elif kind == "stitch":
        c.update(w=_side(rng, 512, 4096), h=_side(rng, 512, 4096))
    else:
        c.update(w=_side(rng, 256, 6144), h=_side(rng, 256, 6144), craters=40)
    return c


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------

def _terrain(w, h, texel, amp, craters, seed):
    """Eight octaves of smooth value noise (wavelengths S, S/2, ... of the longer side S,
    amplitudes halving) plus bowl craters with raised rims; float32 [h, w] metres."""
    g = torch.Generator(device="cpu")
    g.manual_seed(seed)
    S = max(w, h)
    total = sum(0.5 ** o for o in range(8))
    out = torch.zeros((h, w), dtype=torch.float32, device=DEV)
    for o in range(8):
        n = 2 ** o
        ny = max(1, math.ceil(n * h / S))
        nx = max(1, math.ceil(n * w / S))
        lat = (torch.rand((1, 1, ny + 2, nx + 2), generator=g) * 2.0 - 1.0).to(DEV)
        out += F.interpolate(lat, size=(h, w), mode="bicubic", align_corners=True)[0, 0] * (
            amp * 0.5 ** o / total)
    u = torch.rand((3, max(1, craters)), generator=g, dtype=torch.float64).tolist()
    for k in range(craters):
        # cumulative D^-2 law on [50 m, 5 km], at most a third of the tile
        D = min((50.0 ** -2 - u[0][k] * (50.0 ** -2 - 5000.0 ** -2)) ** -0.5, S * texel / 3.0)
        R, xc, yc = 0.5 * D, u[1][k] * w * texel, u[2][k] * h * texel
        i0, i1 = max(0, int((xc - 3 * R) / texel)), min(w, int((xc + 3 * R) / texel) + 2)
        j0, j1 = max(0, int((yc - 3 * R) / texel)), min(h, int((yc + 3 * R) / texel) + 2)
        x = (torch.arange(i0, i1, device=DEV) + 0.5) * texel - xc
        y = (torch.arange(j0, j1, device=DEV) + 0.5) * texel - yc
        r = torch.sqrt(x[None, :] ** 2 + y[:, None] ** 2) / R
        bowl = D * (0.2 * r * r - 0.16)
        flank = 0.04 * D * ((1.0 / r.clamp(min=1.0)) ** 3 - 1.0 / 27.0) * (27.0 / 26.0)
        out[j0:j1, i0:i1] += torch.where(r <= 1.0, bowl, flank.clamp(min=0.0))
    return out.contiguous()


def _rng(seed):
    return random.Random(seed * 7919 + 13)


def _suns(case, seed):
    """(elevation, azimuth, disc radius) of the case's suns."""
    r = _rng(seed)
    a0 = r.uniform(0.0, 2.0 * math.pi)
    if "suns" not in case:
        return [(math.radians(case["elev"]), a0, DISC)]
    n = case["suns"]
    return [(math.radians(0.5 + 2.5 * (k + 0.5) / n), a0 + 0.6 * k, DISC) for k in range(n)]


def _params(case):
    return ss.Params(radius_m=math.inf if case.get("plane") else R_MOON, max_len_m=case["cap"],
                     mode=MODES[case["mode"]], **RUNS[case.get("runs", "geometric")])


def _window(case):
    """The rays' rectangle: the middle half of the tile where the case is a core in its halo."""
    w, h = case["w"], case["h"]
    return (w // 4, h // 4, w // 2, h // 2) if case.get("core") else None


def _tiles(case):
    """(w, h, texel) of a batch's tiles: the named one and smaller, odder ones."""
    out = []
    for k in range(case.get("tiles", 1)):
        out.append((max(64, case["w"] // (k + 1) - 3 * k), max(64, case["h"] // (k + 1) - k),
                    case["texel"] + 2.5 * k))
    return out


def _camera(case):
    """8 km up over the tile's south-west quarter, heading north-east, 25 degrees down."""
    S = case["w"] * case["texel"]
    th = math.tan(math.radians(30.0))
    d, z = math.cos(math.radians(25.0)) / math.sqrt(2.0), -math.sin(math.radians(25.0))
    s2 = 1.0 / math.sqrt(2.0)
    tv = th * case["py"] / case["px"]
    up = (-z * s2 * tv, -z * s2 * tv, math.cos(math.radians(25.0)) * tv)
    return ss.Camera(width=case["px"], height=case["py"], eye=(-0.3 * S, -0.3 * S, 8000.0),
                     fwd=(d, d, z), right=(s2 * th, -s2 * th, 0.0), up=up,
                     step_m=0.5 * case["texel"])


def _image_points(case):
    """Texel coordinates of the points that camera sees on level ground (NaN: sky, or beyond the
    tile): an image of surface points whose neighbours are neighbours on the terrain."""
    cam = _camera(case)
    px = (torch.arange(cam.width, device=DEV, dtype=torch.float64) + 0.5) * (2.0 / cam.width) - 1.0
    py = 1.0 - (torch.arange(cam.height, device=DEV, dtype=torch.float64) + 0.5) * (2.0 / cam.height)
    v = [cam.fwd[k] + px[None, :] * cam.right[k] + py[:, None] * cam.up[k] for k in range(3)]
    t = -cam.eye[2] / v[2]
    q = [(cam.eye[k] + t * v[k]) / case["texel"] + 0.5 * n for k, n in ((0, case["w"]), (1, case["h"]))]
    ok = (v[2] < 0) & (q[0] >= 0) & (q[0] < case["w"]) & (q[1] >= 0) & (q[1] < case["h"])
    xy = torch.stack(q, dim=-1)
    return torch.where(ok[..., None], xy, torch.full_like(xy, math.nan)).float().contiguous()


def _seam_frames(case):
    """Two cube-face sub-tiles meeting at the +z/+x seam and the working tile 1.2 km from it."""
    w, h, D = case["w"], case["h"], case["texel"]
    ns = max(w, h) * 3 // 2
    plane = ns * D
    fa = ss.Frame(ns, ns, D, (0.0, 0.0, 1.0), (1.0, 0.0, 0.0), (0.0, 1.0, 0.0),
                  (R_MOON - 0.5 * plane, 0.0))
    fb = ss.Frame(ns, ns, D, (1.0, 0.0, 0.0), (0.0, 0.0, -1.0), (0.0, 1.0, 0.0),
                  (-R_MOON + 0.5 * plane, 0.0))
    rot = math.pi / 4 + 1.2e3 / R_MOON
    fw = ss.Frame(w, h, D, (math.cos(rot), 0.0, math.sin(rot)), (math.sin(rot), 0.0, -math.cos(rot)),
                  (0.0, 1.0, 0.0))
    return fa, fb, fw


def prepare(case, seed):
    k = case["kind"]
    if k == "stitch":
        fa, fb, fw = _seam_frames(case)
        src = [(_terrain(f.width, f.rows, f.texel_m, case["amp"], 0, seed * 2 + n), f)
               for n, f in enumerate((fa, fb))]
        return dict(kind=k, sources=src, frame=fw)
    if k in ("plan", "batched"):
        tiles = _tiles(case)
        hs = [_terrain(w, h, tx, case["amp"], case["craters"], seed + 1000 * n)
              for n, (w, h, tx) in enumerate(tiles)]
        tx = [t[2] for t in tiles]
        if k == "plan":
            return dict(kind=k, plan=ss.BatchedPlan(hs, tx, _suns(case, seed), _params(case)))
        return dict(kind=k, heights=hs, texels=tx, suns=_suns(case, seed), params=_params(case))
    st = dict(kind=k, h=_terrain(case["w"], case["h"], case["texel"], case["amp"], case["craters"],
                                 seed), texel=case["texel"], w=case["w"], rows=case["h"])
    if k == "terrain":
        return st
    st.update(sun=_suns(case, seed)[0], params=_params(case), window=_window(case))
    if k == "frame":
        # a program that draws frames keeps its terrain's pyramids
        st.update(cam=_camera(case), mm=ss.maxmip(st["h"]), bound=ss.bound_build(st["h"]))
    if k in ("train", "image_train"):
        e, a, r = st["sun"]
        st.update(leaf=st["h"].clone().requires_grad_(True),
                  e=torch.tensor(e, dtype=torch.float64, requires_grad=True),
                  a=torch.tensor(a, dtype=torch.float64, requires_grad=True), r=r,
                  record=case.get("record", False))
        shape = (case["h"], case["w"])
        if k == "image_train":
            st["xy"] = _image_points(case)
            shape = tuple(st["xy"].shape[:2])
        st["g"] = _upstream(shape, seed)
    return st


def _upstream(shape, seed):
    """dL/ds of a training step's loss."""
    g = torch.Generator(device="cpu")
    g.manual_seed(seed + 5)
    base = torch.rand((1, 1, 65, 65), generator=g).to(DEV) + 0.25
    return F.interpolate(base, size=shape, mode="bilinear", align_corners=True)[0, 0].contiguous()


def run(st):
    k = st["kind"]
    if k == "cast":
        return ss.shadow_cast(st["h"], st["texel"], *st["sun"], st["params"], window=st["window"])
    if k == "plan":
        return [o for row in st["plan"].launch() for o in row]
    if k == "batched":
        outs = ss.shadow_cast_batched(st["heights"], st["texels"], st["suns"], st["params"])
        return [o for row in outs for o in row]
    if k == "train":
        s = ss.shadow(st["leaf"], st["e"], st["a"], st["texel"], st["r"], st["params"],
                      record=st["record"])
        gh, ge, ga = torch.autograd.grad(s, [st["leaf"], st["e"], st["a"]], st["g"])
        return [s, gh, ge, ga]
    if k == "image_train":
        s = ss.shadow_at(st["leaf"], st["e"], st["a"], st["xy"], st["texel"], st["r"], st["params"])
        gh, ge, ga = torch.autograd.grad(s, [st["leaf"], st["e"], st["a"]], st["g"])
        return [s, gh, ge, ga]
    if k == "frame":
        return list(ss.frame(st["h"], st["texel"], st["cam"], *st["sun"], st["params"], st["mm"],
                             st["bound"]))
    if k == "stitch":
        return ss.stitch(st["sources"], st["frame"], R_MOON)
    mm = ss.maxmip(st["h"])
    bound = ss.bound_build(st["h"])
    return ss.maxmip_unpack(mm, st["w"], st["rows"]) + ss.bound_unpack(bound, st["w"], st["rows"])


# ---------------------------------------------------------------------------
# Work: inputs read once, outputs written once; operations per ray as the formulas count them
# ---------------------------------------------------------------------------

# operations a ray cannot do without, by mode: about 45 bounds of 35 operations and 10 samples of
# 45 for the descent; 31 evaluations for three point-sample runs; the steps that remain after the
# early exits for stepping; the walk's 62 tests and 19 samples in the exact mode
_OPS = {"descent": 45 * 35 + 10 * 45, "point": 31 * 35, "exact": 62 * 35 + 19 * 45}


def _ray_ops(case):
    if case["mode"] == "uniform":
        return 40.0 * 0.2 * max(case["w"], case["h"])
    return float(_OPS[case["mode"]])


def work(case):
    k = case["kind"]
    if k == "stitch":
        n = case["w"] * case["h"]
        return dict(bytes=8.0 * n, flops=60.0 * n)
    if k in ("plan", "batched"):
        n = sum(w * h for w, h, _ in _tiles(case))
        rays = n * case["suns"]
        return dict(bytes=4.0 * (n + rays), flops=rays * _ray_ops(case))
    n = case["w"] * case["h"]
    if k == "terrain":
        return dict(bytes=4.0 * n * (1.0 + 1.0 / 3.0 + 4.0 / 3.0), flops=12.0 * n)
    if k == "frame":
        pix = case["px"] * case["py"]
        return dict(bytes=4.0 * n + 16.0 * pix, flops=pix * (10.0 * 60.0 + 0.5 * _ray_ops(case)))
    if k == "image_train":
        pix = case["px"] * case["py"]
        return dict(bytes=8.0 * n + 16.0 * pix, flops=pix * (1.3 * _ray_ops(case)))
    w = _window(case)
    rays = w[2] * w[3] if w else n
    if k == "train":
        return dict(bytes=16.0 * n, flops=rays * 1.3 * _ray_ops(case))
    return dict(bytes=4.0 * (n + rays), flops=rays * _ray_ops(case))


# ---------------------------------------------------------------------------
# The same definitions in float64
# ---------------------------------------------------------------------------

def _levels(h):
    """h and its maximum mipmap (ceil-halving), float32 (a maximum rounds nothing)."""
    out = [h]
    while max(out[-1].shape) > 1:
        out.append(F.max_pool2d(out[-1][None, None], 2, ceil_mode=True)[0, 0])
    return out


class _Scene:
    def __init__(self, h, texel, sun, params):
        self.h, self.texel, self.p = h, texel, params
        self.lv = _levels(h)
        self.H, self.W = h.shape
        self.R = params.radius_m
        self.sphere = not math.isinf(self.R)
        e, a, self.rL = sun
        self.L = (math.cos(e) * math.cos(a), math.cos(e) * math.sin(a), math.sin(e))
        self.half = 0.5 * texel / math.cos(e)
        self.top = float(h.max())
        # the concatenated runs: (top level, first half-texel grid index)
        diag = math.hypot(self.W, self.H) + 2.0
        need = params.max_len_m / texel if params.max_len_m > 0 else diag
        self.runs, ga, done, j = [], 0, 0.0, 0
        while True:
            n = params.n_prime0 + (j if params.schedule == ss.SS_SCHED_GEOMETRIC else 0)
            if params.schedule == ss.SS_SCHED_LIST:
                n = params.n_prime_list[j]
            m = max(1, min(n, len(self.lv))) - 1
            self.runs.append((m, ga))
            ga += 2 << m
            done += 2.0 ** m
            j += 1
            if (j >= params.n_segments) if params.n_segments > 0 else (done >= need):
                break
        self.end = (ga + 1) * self.half
        self.cap = params.max_len_m / texel * 2.0 * self.half if params.max_len_m > 0 else self.end

    def tau(self, j):
        return (self.runs[j][1] + 1) * self.half if j < len(self.runs) else self.end


class _Rays:
    """Rays from texel coordinates (x, y) on the terrain of height z0; fields are float64 [n]."""

    def __init__(self, S, x, y, z0):
        self.S, self.x, self.y, self.z0 = S, x, y, z0
        Lx, Ly, Lz = S.L
        if S.sphere:
            a = (x - 0.5 * S.W) * S.texel / S.R
            b = (y - 0.5 * S.H) * S.texel / S.R
            g = torch.sqrt(1.0 + a * a + b * b)
            r1 = 1.0 + z0 / S.R
            self.sp = (a * Lx + b * Ly + Lz) / g
            self.cp = torch.sqrt((b * Lz - Ly) ** 2 + (Lx - a * Lz) ** 2 + (a * Ly - b * Lx) ** 2) / g
            k = g / (r1 * S.texel)
            self.Kx, self.Ky = (Lx - a * Lz) * k, (Ly - b * Lz) * k
            self.c = Lz * g / (r1 * S.R)
            self.ir = 1.0 / (S.R * r1)
            th = -self.sp / self.ir
            self.umin = torch.where(self.sp < 0, th / (1.0 + self.c * th),
                                    torch.full_like(th, -math.inf))
        else:
            o = torch.ones_like(x)
            self.sp, self.cp = Lz * o, (Lx * Lx + Ly * Ly) ** 0.5 * o
            self.Kx, self.Ky = Lx / S.texel * o, Ly / S.texel * o
            self.c, self.ir = 0.0 * o, 0.0 * o
            self.umin = (-math.inf if Lz >= 0 else math.inf) * o
        inf = torch.full_like(x, math.inf)
        ux = torch.where(self.Kx > 0, (S.W - x) / self.Kx, torch.where(self.Kx < 0, -x / self.Kx, inf))
        uy = torch.where(self.Ky > 0, (S.H - y) / self.Ky, torch.where(self.Ky < 0, -y / self.Ky, inf))
        self.uexit = torch.minimum(ux, uy)

    def at(self, idx):
        r = object.__new__(_Rays)
        r.S = self.S
        for n, v in self.__dict__.items():
            if n != "S":
                setattr(r, n, v[idx])
        return r

    def u(self, t):
        return t / (1.0 + self.c * t)

    def t(self, u):
        return u / (1.0 - self.c * u)

    def rise(self, t):
        q = t * self.ir
        q2 = 2.0 * self.sp + q
        return t * q2 / (torch.sqrt(1.0 + q * q2) + 1.0) + self.z0

    def key(self, t, dh):
        """Tangent of the angle between the sun and the terrain point below the ray's tip."""
        q = t * self.ir
        num = dh * self.cp
        den = t * torch.sqrt(1.0 + q * (2.0 * self.sp + q)) - dh * (self.sp + q)
        inf = torch.full_like(num, math.inf)
        return torch.where(den > 0, num / den, torch.where(num >= 0, inf, -inf))

    def ground(self, t, h=None):
        """Bilinear terrain below the tip, and dh = the tip's height above it."""
        S, u = self.S, self.u(t)
        return _bilinear(S.h if h is None else h, self.x + self.Kx * u, self.y + self.Ky * u)

    def clears(self, t, key):
        """Nothing at ray length >= t can matter: the highest terrain already clears
        min(angle, disc radius), with room to spare."""
        S = self.S
        top = torch.maximum(torch.full_like(self.z0, S.top), self.z0)
        d = self.rise(t) - top
        need = torch.tan(torch.atan(key).clamp(max=S.rL) + 1e-6)
        return (d > 0) & (self.key(t, d) >= need)


def _bilinear(h, qx, qy):
    H, W = h.shape
    x, y = qx - 0.5, qy - 0.5
    x0, y0 = torch.floor(x), torch.floor(y)
    fx, fy = x - x0, y - y0
    xa, xb = x0.long().clamp(0, W - 1), (x0.long() + 1).clamp(0, W - 1)
    ya, yb = y0.long().clamp(0, H - 1), (y0.long() + 1).clamp(0, H - 1)
    f = h.reshape(-1)
    return ((1 - fy) * ((1 - fx) * f[ya * W + xa].double() + fx * f[ya * W + xb].double())
            + fy * ((1 - fx) * f[yb * W + xa].double() + fx * f[yb * W + xb].double()))


def _texel(S, m, cx, cy):
    """Level-m maxima at integer texels, and whether they lie in the level."""
    L = S.lv[m]
    hh, ww = L.shape
    ok = (cx >= 0) & (cy >= 0) & (cx < ww) & (cy < hh)
    return L.reshape(-1)[cy.clamp(0, hh - 1) * ww + cx.clamp(0, ww - 1)].double(), ok


def _run_descent(S, r, j):
    """One run: the texels the ray crosses at the top level, the smallest lower bound (farthest
    on ties), its crossed children down to level 0, three samples.  -> (key, n, found)"""
    m, _ = S.runs[j]
    inf = torch.full_like(r.x, math.inf)
    ua = r.u(torch.full_like(r.x, S.tau(j)))
    ub = torch.minimum(r.u(torch.full_like(r.x, S.tau(j + 1))), r.uexit)
    fx_, fy_ = r.Kx >= 0, r.Ky >= 0

    def cross(gx, gy):
        return (torch.where(r.Kx != 0, (gx - r.x) / r.Kx, inf),
                torch.where(r.Ky != 0, (gy - r.y) / r.Ky, inf))

    def low(u0, u1):
        uc = torch.minimum(torch.maximum(r.umin, u0), u1)
        return r.rise(r.t(uc))

    T = float(1 << m)
    cx = torch.floor((r.x + r.Kx * ua) / T).long()
    cy = torch.floor((r.y + r.Ky * ua) / T).long()
    best, bx, by, b0, b1 = inf, cx, cy, ua, ua
    u0, live = ua, torch.ones_like(fx_)
    for _ in range(8):
        gx, gy = cross((cx + fx_.long()).double() * T, (cy + fy_.long()).double() * T)
        u1 = torch.minimum(torch.minimum(gx, gy), ub)
        M, ok = _texel(S, m, cx, cy)
        lb = low(u0, u1) - M
        take = live & ok & (u1 > u0) & (lb <= best)
        best, b0, b1 = torch.where(take, lb, best), torch.where(take, u0, b0), torch.where(take, u1, b1)
        bx, by = torch.where(take, cx, bx), torch.where(take, cy, by)
        u0 = torch.maximum(u0, u1)
        live = live & (u1 < ub)
        if not bool(live.any()):
            break
        cx = cx + torch.where(gx <= gy, torch.sign(r.Kx), 0.0).long()
        cy = cy + torch.where(gy <= gx, torch.sign(r.Ky), 0.0).long()
    found = best < math.inf
    for lv in range(m, 0, -1):
        half = float(1 << (lv - 1))
        px, py = 2 * bx, 2 * by
        ux, uy = cross((px + 1).double() * half, (py + 1).double() * half)
        first = ux <= uy
        c1 = torch.minimum(torch.maximum(torch.minimum(ux, uy), b0), b1)
        c2 = torch.minimum(torch.maximum(torch.maximum(ux, uy), b0), b1)
        xa, ya = px + (~fx_).long(), py + (~fy_).long()
        xc, yc = px + fx_.long(), py + fy_.long()
        cand = [(xa, ya, b0, c1), (torch.where(first, xc, xa), torch.where(first, ya, yc), c1, c2),
                (xc, yc, c2, b1)]
        best = inf
        nx, ny, n0, n1 = bx, by, b0, b1
        for x, y, lo, hi in cand:
            M, ok = _texel(S, lv - 1, x, y)
            lb = torch.where(ok & (hi > lo), low(lo, hi) - M, inf)
            take = (lb <= best) & (lb < math.inf)
            best = torch.where(take, lb, best)
            nx, ny = torch.where(take, x, nx), torch.where(take, y, ny)
            n0, n1 = torch.where(take, lo, n0), torch.where(take, hi, n1)
        bx, by, b0, b1 = nx, ny, n0, n1
        found = found & (best < math.inf)
    mid = 0.5 * (r.t(b0) + r.t(b1))
    nc = torch.floor((mid - S.half) / S.half + 0.5)
    return _three(S, r, [nc - 1, nc, nc + 1], found, far_first=False)


def _three(S, r, ns, found, far_first):
    """The smallest of three samples by height above the terrain, and its clearance."""
    bdh = torch.full_like(r.x, math.inf)
    bn = torch.zeros_like(r.x)
    for n in ns:
        t = (n + 1.0) * S.half
        t1 = t.clamp(min=S.half)
        dh = r.rise(t1) - r.ground(t1)
        ok = (n >= 0) & (r.u(t1) < r.uexit)
        take = ok & ((dh < bdh) if far_first else (dh <= bdh))
        bdh, bn = torch.where(take, dh, bdh), torch.where(take, n, bn)
    found = found & (bdh < math.inf)
    return r.key((bn + 1.0) * S.half, bdh), bn.long(), found


def _run_point(S, r, j):
    """One run of the point-sample descent (far to near, strict minimum)."""
    m0, a = S.runs[j]
    K = torch.full_like(r.x, float(2 << m0))
    found = torch.ones_like(r.x, dtype=torch.bool)
    for m in range(m0, 0, -1):
        best = torch.full_like(r.x, math.inf)
        ks = torch.full_like(r.x, -1.0)
        for q in range(3):
            kk = K - q * (1 << m)
            t = (a + kk + 1.0) * S.half
            u = r.u(t)
            cx = torch.floor(r.x + r.Kx * u).long() >> m
            cy = torch.floor(r.y + r.Ky * u).long() >> m
            M, ok = _texel(S, m, cx, cy)
            v = r.rise(t) - M
            take = ok & (u < r.uexit) & (v < best)
            best, ks = torch.where(take, v, best), torch.where(take, kk, ks)
        found = found & (ks >= 0)
        K = torch.where(ks >= 0, ks, K) + (1 << m)
    return _three(S, r, [a + K, a + K - 1, a + K - 2], found, far_first=True)


def _trace(S, r):
    """(key, n): the smallest clearance tangent over the ray and its sample's index."""
    n_rays = r.x.numel()
    key = torch.full_like(r.x, math.inf)
    num = torch.full((n_rays,), -1, dtype=torch.long, device=r.x.device)
    idx = torch.arange(n_rays, device=r.x.device)
    mode = S.p.mode
    umbra = -math.tan(S.rL)
    if mode in (ss.SS_MODE_DP, ss.SS_MODE_POINT):
        for j in range(len(S.runs)):
            t0 = torch.full_like(r.x, S.tau(j))
            lo = max(S.half, S.tau(j) - 1.5 * S.half)
            keep = (r.u(t0) < r.uexit) & (key[idx] > umbra) & ~r.clears(torch.full_like(r.x, lo), key[idx])
            sel = keep.nonzero()[:, 0]
            if sel.numel() == 0:
                break
            r, idx = r.at(sel), idx[sel]
            k, n, ok = (_run_descent if mode == ss.SS_MODE_DP else _run_point)(S, r, j)
            take = ok & (k < key[idx])
            key[idx] = torch.where(take, k, key[idx])
            num[idx] = torch.where(take, n, num[idx])
        return key, num
    step = S.half if mode == ss.SS_MODE_EXACT else S.p.uniform_step * 2.0 * S.half
    best, bn = key.clone(), num.clone()
    k = 0
    while True:
        t = S.half + k * step
        tt = torch.full_like(r.x, t)
        if k % 16 == 0:
            keep = (r.u(tt) < r.uexit) & (best > umbra) & ~r.clears(tt, best)
            sel = keep.nonzero()[:, 0]
            gone = (~keep).nonzero()[:, 0]
            key[idx[gone]], num[idx[gone]] = best[gone], bn[gone]
            if sel.numel() == 0 or t > S.cap:
                key[idx], num[idx] = best, bn
                return key, num
            r, idx, best, bn = r.at(sel), idx[sel], best[sel], bn[sel]
            tt = tt[sel]
        if t <= S.cap:
            c = r.key(tt, r.rise(tt) - r.ground(tt))
            take = (r.u(tt) < r.uexit) & (c < best)
            best = torch.where(take, c, best)
            bn = torch.where(take, torch.full_like(bn, k), bn)
        k += 1


def _disc(key, rL):
    d = (torch.atan(key) / rL).clamp(-1.0, 1.0)
    v = (math.pi - torch.acos(d) + d * torch.sqrt((1.0 - d * d).clamp(min=0.0))) / math.pi
    return torch.where(d >= 1.0, torch.ones_like(v), torch.where(d <= -1.0, torch.zeros_like(v), v))


def _shade(S, x, y):
    """s and the deciding sample for origins at texel coordinates x, y (flat), in pieces."""
    s, n = [], []
    for k in range(0, x.numel(), 1 << 22):
        xs, ys = x[k:k + (1 << 22)], y[k:k + (1 << 22)]
        key, num = _trace(S, _Rays(S, xs, ys, _bilinear(S.h, xs, ys)))
        s.append(_disc(key, S.rL))
        n.append(num)
    return torch.cat(s), torch.cat(n)


def _centres(w, h, window):
    x0, y0, rw, rh = window or (0, 0, w, h)
    x = torch.arange(x0, x0 + rw, device=DEV, dtype=torch.float64) + 0.5
    y = torch.arange(y0, y0 + rh, device=DEV, dtype=torch.float64) + 0.5
    return x.repeat(rh), y.repeat_interleave(rw), (rh, rw)


def _gradients(S, sun, x, y, n, s, g):
    """dL/dh and dL/d(elevation, azimuth) through each ray's deciding sample, by autograd."""
    idx = ((n >= 0) & (s > 0) & (s < 1) & (g != 0)).nonzero()[:, 0]
    x, y, n, g = x[idx], y[idx], n[idx].double(), g[idx].double()
    h = S.h.double().requires_grad_(True)
    e = torch.tensor(sun[0], dtype=torch.float64, device=DEV, requires_grad=True)
    a = torch.tensor(sun[1], dtype=torch.float64, device=DEV, requires_grad=True)
    D = object.__new__(_Scene)
    D.__dict__.update(S.__dict__)
    D.L = (torch.cos(e) * torch.cos(a), torch.cos(e) * torch.sin(a), torch.sin(e))
    D.half = 0.5 * S.texel / torch.cos(e)
    r = _Rays(D, x, y, _bilinear(h, x, y))
    step = D.half * (2.0 * S.p.uniform_step if S.p.mode == ss.SS_MODE_UNIFORM else 1.0)
    t = D.half + n * step
    d = torch.atan(r.key(t, r.rise(t) - r.ground(t, h))) / S.rL
    d = d.clamp(-1.0, 1.0)
    v = (math.pi - torch.acos(d) + d * torch.sqrt((1.0 - d * d).clamp(min=1e-300))) / math.pi
    return torch.autograd.grad((v * g).sum(), [h, e, a])


def _exact_stitch(sources, fd):
    out = torch.full((fd.rows, fd.width), math.nan, dtype=torch.float64, device=DEV)
    X = fd.origin[0] + (torch.arange(fd.width, device=DEV, dtype=torch.float64) + 0.5 - 0.5 * fd.width) * fd.texel_m
    Y = fd.origin[1] + (torch.arange(fd.rows, device=DEV, dtype=torch.float64) + 0.5 - 0.5 * fd.rows) * fd.texel_m
    for h, f in sources:
        P = [R_MOON * fd.centre[k] + X[None, :] * fd.ex[k] + Y[:, None] * fd.ey[k] for k in range(3)]
        dot = lambda v: P[0] * v[0] + P[1] * v[1] + P[2] * v[2]  # noqa: E731
        z = dot(f.centre)
        qx = (R_MOON / z * dot(f.ex) - f.origin[0]) / f.texel_m + 0.5 * f.width
        qy = (R_MOON / z * dot(f.ey) - f.origin[1]) / f.texel_m + 0.5 * f.rows
        ok = (z > 0) & (qx >= 0) & (qx < f.width) & (qy >= 0) & (qy < f.rows)
        v = _bilinear(h, qx.clamp(0, f.width), qy.clamp(0, f.rows))
        out = torch.where(ok, v, out)
    return out


def exact(case, seed):
    k = case["kind"]
    if k == "frame":
        # a view ray's hit is the first grid sample below the terrain: at a grazing hit rounding
        # decides between this sample, a later one and none, so there is no single value
        return None
    if k == "stitch":
        st = prepare(case, seed)
        return _exact_stitch(st["sources"], st["frame"])
    if k in ("plan", "batched"):
        tiles, suns, p = _tiles(case), _suns(case, seed), _params(case)
        if sum(w * h for w, h, _ in tiles) * len(suns) > LIMIT_RAYS:
            return None
        out = []
        for n, (w, h, tx) in enumerate(tiles):
            t = _terrain(w, h, tx, case["amp"], case["craters"], seed + 1000 * n)
            for sun in suns:
                x, y, shape = _centres(w, h, None)
                out.append(_shade(_Scene(t, tx, sun, p), x, y)[0].view(shape))
        return out
    h = _terrain(case["w"], case["h"], case["texel"], case["amp"], case["craters"], seed)
    if k == "terrain":
        pad = F.max_pool2d(h[None, None], 3, stride=1, padding=1)[0, 0]
        return [v.double() for v in _levels(h)[1:]] + [v.double() for v in _levels(pad)]
    sun, p = _suns(case, seed)[0], _params(case)
    S = _Scene(h, case["texel"], sun, p)
    if k == "image_train":
        xy = _image_points(case).double()
        shape = tuple(xy.shape[:2])
        x, y = xy[..., 0].reshape(-1), xy[..., 1].reshape(-1)
        sees = (x == x).nonzero()[:, 0]
        s = torch.full((x.numel(),), math.nan, dtype=torch.float64, device=DEV)
        sv, n = _shade(S, x[sees], y[sees])
        s[sees] = sv
        g = _upstream(shape, seed).reshape(-1)[sees]
        gh, ge, ga = _gradients(S, sun, x[sees], y[sees], n, sv, g)
        return [s.view(shape), gh, ge.cpu(), None]
    x, y, shape = _centres(case["w"], case["h"], _window(case))
    if x.numel() > LIMIT_RAYS:
        return None
    s, n = _shade(S, x, y)
    if k == "cast":
        return s.view(shape)
    # the azimuth's gradient is a sum of signed terms that cancel: it has no digits to compare
    gh, ge, _ = _gradients(S, sun, x, y, n, s, _upstream(shape, seed).reshape(-1))
    return [s.view(shape), gh, ge.cpu(), None]
