"""What a user of the renderer has it do, as measurable cases.

Every case is one program: stacks of jet-like epochs resident on the device
(emissivity with lognormal turbulence, matter at rest outside a relativistic
spine and its knots), views around them, and one call (or one short sequence of
calls) through the package's public entry points.  The sizes are those of the
benchmark's workloads and of the tests, or spread around them.

Kinds:
  single    dart_render: one image from one stack
  batch     dart_render_batch: the same views again and again (the plan replays)
  frames    a light curve: successive dart_render_batch calls at other t_obs
  serve     dart_submit / dart_wait: a burst of requests over several stacks
  vector    dart_render_batch on a three-component (I, Q, U) vector stack
  labelled  dart_render_batch on a grid whose core is refined twice
  stream    dart_streamer_render: epochs that are not resident
  refill    dart_stack_set_epochs into a resident stack, a render of it, and
            dart_stack_read_epoch
"""
import math
import random

import numpy as np
import torch

import paper_2609_09322_amd as dart

STORE = {"f64": dart.DART_F64, "f32": dart.DART_F32, "f16": dart.DART_F16, "bf16": dart.DART_BF16}
RECORD = {"f64": 32, "f32": 16, "f16": 8, "bf16": 8}
FLAGS = {"": 0, "nearest": dart.DART_NEAREST_EPOCH, "exact": dart.DART_EXACT_TIME,
         "nolook": dart.DART_NO_LOOKBACK, "force64": dart.DART_FORCE_F64_DDA}
DEFAULT_TUNING = "32,2,8,0,1,0,4"  # the library's own launch shape
ALPHA = 0.6


def _case(name, kind, store, dims, epochs, sides, orient="iso", options="", brick="",
          tuning=DEFAULT_TUNING, frames=0):
    return {"name": name, "kind": kind, "store": store, "nx": dims[0], "ny": dims[1],
            "nz": dims[2], "epochs": epochs, "sides": ",".join(str(s) for s in sides),
            "orient": orient, "options": options, "brick": brick, "tuning": tuning,
            "frames": frames}


def listed():
    return [
        # The smallest call: the 64^3 FP64 stack of the smoke check, one 128^2
        # image to the host with flux and cell-steps.  Latency.
        _case("smoke_f64", "single", "f64", (64, 64, 64), 4, [128], options="stats"),
        # One image of a mid-size FP32 jet without any tuning: interactive use.
        _case("single_f32", "single", "f32", (128, 128, 256), 8, [512]),
        # The benchmark's headline: four 512^2 views of the FP32 jet, at the
        # bricks and launch shape that dart_autotune finds for it.
        _case("jet_f32", "batch", "f32", (256, 256, 512), 16, [512] * 4, orient="jet",
              brick="1,16,2", tuning="64,1,8,0,0,0,8"),
        # The benchmark's uneven FP16 batch: 64 isotropic views from 128^2 to
        # 1024^2, tuned.  Throughput.
        _case("uneven_f16", "batch", "f16", (384, 384, 384), 32,
              [128, 256, 512, 1024] * 16, brick="1,2,8", tuning="16,4,16,0,1,6,8"),
        # A slab of the benchmark's largest grid in BF16 with FP64 ray
        # parameters (its plane is addressed by 64 bits), 1024^2 views, tuned.
        _case("slab_bf16", "batch", "bf16", (512, 512, 1024), 10, [1024] * 8,
              options="force64", brick="1,2,16", tuning="16,4,8,4,1,0,8"),
        # The reference precision with the marching options, as a parity check
        # or a convergence study renders them; images, flux and steps.
        _case("options_f64", "batch", "f64", (128, 128, 128), 6, [256] * 4,
              options="exact,nearest,,nolook,stats"),
        # Serving: a burst of requests of all sizes over three FP16 stacks.
        _case("serve_f16", "serve", "f16", (128, 128, 128), 8,
              [128, 256, 512, 1024] * 6, brick="1,8,2", tuning="8,8,12,0,1,6,8"),
        # A light curve of a small odd-sized FP16 grid: other views every call,
        # without tuning.  Planning and launches count as much as marching.
        _case("frames_f16", "frames", "f16", (150, 97, 211), 6, [136, 200], frames=10),
        # Polarised components (I, Q, U) integrated in one march, FP32.
        _case("vector_f32", "vector", "f32", (128, 128, 256), 8, [512] * 2, brick="1,8,1",
              tuning="64,1,12,0,1,0,8"),
        # Multi-resolution domain: six coarse blocks around a core refined twice.
        _case("labelled_f32", "labelled", "f32", (128, 128, 256), 8, [512] * 4, orient="jet",
              brick="1,8,1", tuning="64,1,12,0,1,0,8"),
        # Out-of-core: every epoch passes through the ring, from device arrays
        # in the caller's layout (a simulation on the same GPU).
        _case("stream_f32", "stream", "f32", (192, 192, 256), 10, [512] * 2, orient="jet"),
        # A running simulation replaces one epoch, looks at the result and
        # reads the epoch back as stored.
        _case("refill_f16", "refill", "f16", (256, 256, 256), 8, [256] * 2),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["single", "single", "batch", "batch", "batch", "frames", "serve", "vector",
                       "labelled", "stream", "refill"])
    store = rng.choice(["f32", "f16", "bf16", "f64"])
    if kind == "serve" and store == "f64":
        store = "f32"
    hi = {"batch": 384, "serve": 144}.get(kind, 224)
    dims = [_log(rng, 24, hi) for _ in range(3)]
    if kind == "labelled":
        dims = [max(8, d // 4) * 4 for d in dims]
    epochs = _log(rng, 2, 24)
    # (what the case holds: the served stacks are up to 8 times the grid)
    share = {"serve": 21, "vector": 4, "stream": 4, "labelled": 3}.get(kind, 1)
    while dims[0] * dims[1] * dims[2] * epochs * RECORD[store] * share > (8 << 30):
        epochs = max(1, epochs // 2)
    n = {"single": 1, "batch": _log(rng, 1, 24), "serve": _log(rng, 1, 24)}.get(kind, rng.randint(1, 4))
    top = 1024 if kind in ("single", "batch") else 512
    sides = [_log(rng, 33, top) for _ in range(n)]
    options = ""
    if kind in ("single", "batch", "frames"):
        options = rng.choice(["", "", "", "nearest", "exact", "nolook", "force64", "stats"])
    brick, tuning = "", DEFAULT_TUNING
    if kind in ("batch", "vector", "serve") and rng.random() < 0.6:
        brick = rng.choice(["1,8,1", "1,16,2", "2,2,2", "1,2,8", "1,4,4", "4,2,2"])
        tuning = rng.choice(["64,1,8,0,0,0,8", "16,4,16,0,1,6,8", "8,8,12,1,1,6,8",
                             "64,1,12,3,1,0,8", "16,4,8,4,1,0,8"])
    c = _case("", kind, store, dims, epochs, sides, options=options, brick=brick, tuning=tuning,
              frames=rng.randint(2, 12) if kind == "frames" else 0)
    del c["name"]
    return c


# ---------------------------------------------------------------------- inputs

def _times(dims, epochs):
    """Epochs over the light-crossing time of the grid's diagonal, so that at
    t_obs = 0 every cell lies inside the coverage."""
    L = math.sqrt(sum(float(d) ** 2 for d in dims))
    if epochs == 1:
        return np.zeros(1)
    return -0.5 * L + np.arange(epochs) * (L / (epochs - 1))


def _held(x, store):
    """x at the storage type's values, so that the stored stack is the input."""
    if store == "f16":
        return x.half().to(x.dtype)
    if store == "bf16":
        return x.bfloat16().to(x.dtype)
    return x


class _Jet:
    """Epochs of a jet along z: lognormal turbulence advected along the axis, a
    spine whose Lorentz factor falls outward, knots, and matter at rest around
    (a hundredth of the emissivity)."""

    def __init__(self, dims, epochs, store, seed):
        self.dims, self.store = dims, store
        self.times = _times(dims, epochs)
        g = torch.Generator(device="cuda").manual_seed(int(seed) * 7919 + 11)
        nx, ny, nz = dims
        low = [max(2, d // 6) for d in (nz, ny, nx)]
        noise = torch.randn([1, 1] + low, generator=g, device="cuda")
        noise = torch.nn.functional.interpolate(noise, size=(nz, ny, nx), mode="trilinear",
                                                align_corners=False)[0, 0]
        self.rho = torch.exp(1.1 * noise - 0.2)
        del noise
        self.radius = max(2.5, 12.0 * min(nx, ny) / 256.0)
        x = torch.arange(nx, device="cuda") + 0.5 - 0.5 * nx
        y = torch.arange(ny, device="cuda") + 0.5 - 0.5 * ny
        self.r2 = (x[None, :] ** 2 + y[:, None] ** 2)[None]
        rel = (self.r2 / self.radius ** 2).clamp(max=1.0)
        self.inside = (self.r2 <= self.radius ** 2).float()
        gamma = 1.2 + 3.8 * (1.0 - rel)
        self.spine = torch.sqrt(1.0 - 1.0 / gamma ** 2) * self.inside
        self.env = 0.01 + 0.99 * self.inside
        rng = random.Random(int(seed) * 31 + 5)
        self.knots = [rng.uniform(0.0, nz) for _ in range(4)]
        self.z = torch.arange(nz, device="cuda") + 0.5

    def epoch(self, m):
        """(j [nz][ny][nx], beta [nz][ny][nx][3]) of epoch m, float32 (float64
        for an FP64 stack)."""
        t = float(self.times[m])
        j = torch.roll(self.rho, int(round(0.5 * t)), 0) * self.env
        bz = self.spine.expand_as(j).clone()
        near = torch.zeros_like(self.z)
        for z0 in self.knots:
            near = torch.maximum(near, torch.exp(-(self.z - (z0 + 0.98 * t)) ** 2
                                                 / (0.5 * self.radius ** 2)))
        j *= 1.0 + 4.0 * near[:, None, None] * torch.exp(-self.r2 / (0.5 * self.radius ** 2))
        bz = torch.where((near > 0.14)[:, None, None] & (self.inside > 0), 0.98, bz)
        beta = torch.zeros(j.shape + (3,), device="cuda")
        beta[..., 2] = bz
        beta[..., 0] = 0.05 * bz
        out = _held(j, self.store), _held(beta, self.store)
        return tuple(o.double() for o in out) if self.store == "f64" else out

    def load(self, dims=None, cell=(1.0, 1.0, 1.0), of=None):
        """A resident stack of every epoch (of: what to make of each)."""
        s = dart.dart_stack_create(dims or self.dims, cell, self.times, STORE[self.store])
        for m in range(len(self.times)):
            j, b = self.epoch(m) if of is None else of(*self.epoch(m))
            dart.dart_stack_set_epochs(s, m, j[None].contiguous(), b[None].contiguous())
        return s


def _dims(case):
    return case["nx"], case["ny"], case["nz"]


def _sides(case):
    return [int(s) for s in case["sides"].split(",")]


def _options(case, n):
    """(flags of each view, whether flux and steps are asked for)."""
    names = case["options"].split(",") if case["options"] else [""]
    stats = names[-1] == "stats"
    names = names[:-1] if stats else names
    names = names or [""]
    return [FLAGS[names[i % len(names)]] for i in range(n)], stats


def _views(case, seed, t_obs=0.0):
    sides, dims = _sides(case), _dims(case)
    flags, _ = _options(case, len(sides))
    L = math.sqrt(sum(float(d) ** 2 for d in dims))
    rng = random.Random(int(seed) * 17 + 3)
    out_t = dart.DART_F64 if case["store"] == "f64" else dart.DART_F32
    views = []
    for i, p in enumerate(sides):
        th = math.degrees(math.acos(rng.uniform(-1.0, 1.0)))
        ph = rng.uniform(0.0, 360.0)
        if case["orient"] == "jet":  # the headline's inclinations
            th, ph = (10.0, 30.0, 60.0, 90.0)[i % 4], 0.0
        views.append(dart.View(th, ph, p, p, L / p, t_obs, ALPHA, flags[i], out_t))
    return views


def _images(case, views, channels=0):
    t = torch.float64 if case["store"] == "f64" else torch.float32
    lead = (channels,) if channels else ()
    return [torch.zeros(lead + (v.height, v.width), dtype=t, device="cuda") for v in views]


def _tune(case):
    dart.dart_set_tuning(*[int(x) for x in case["tuning"].split(",")])


def _lay(case, stack):
    if case["brick"]:
        dart.dart_stack_rebrick(stack, [int(x) for x in case["brick"].split(",")])
    return stack


def _boxes(dims):
    """Six coarse boxes around the core, and the core: ((x0, x1), (y0, y1), (z0, z1))."""
    nx, ny, nz = dims
    x0, x1, y0, y1, z0, z1 = nx // 4, 3 * nx // 4, ny // 4, 3 * ny // 4, nz // 3, 2 * nz // 3
    X, Y, Z = (0, nx), (0, ny), (z0, z1)
    return [(X, Y, (0, z0)), (X, Y, (z1, nz)), ((0, x0), Y, Z), ((x1, nx), Y, Z),
            ((x0, x1), (0, y0), Z), ((x0, x1), (y1, ny), Z)], ((x0, x1), (y0, y1), Z)


def _cut(box, j, b):
    (x0, x1), (y0, y1), (z0, z1) = box
    return j[z0:z1, y0:y1, x0:x1], b[z0:z1, y0:y1, x0:x1]


def _fine(j, b):
    for d in range(3):
        j, b = j.repeat_interleave(2, dim=d), b.repeat_interleave(2, dim=d)
    return j, b


QU = (lambda j: j, lambda j: 0.5 * j * torch.cos(torch.log1p(j)),
      lambda j: 0.5 * j * torch.sin(torch.log1p(j)))

SERVED = ((1, 1), (1, 4), (2, 2))  # (grid scale, epoch scale) of the served stacks


class _Serving:
    """A running server, stopped with the program that holds it."""

    def __init__(self, n):
        self.srv = dart.dart_server_create(192 << 20, 256, 3)

    def __del__(self):
        if self.srv.handle:
            dart.dart_server_destroy(self.srv)


def prepare(case, seed):
    _tune(case)
    dims, kind, store = _dims(case), case["kind"], case["store"]
    views = _views(case, seed)
    st = {"case": case, "views": views, "stream": torch.cuda.Stream(),
          "stats": _options(case, 1)[1]}
    if kind == "serve":
        rng = random.Random(int(seed) + 41)
        st["stacks"] = [_lay(case, _Jet(tuple(d * g for d in dims), min(32, case["epochs"] * e),
                                        store, seed + k).load())
                        for k, (g, e) in enumerate(SERVED)]
        st["ask"] = []
        for v in views:
            k = rng.randrange(len(SERVED))
            v.pixel_scale *= SERVED[k][0]
            st["ask"].append((st["stacks"][k], v))
        st["images"] = _images(case, views)
        st["server"] = _Serving(len(views))
    elif kind == "vector":
        jet = _Jet(dims, case["epochs"], store, seed)
        st["stack"] = dart.dart_vector_create(
            [_lay(case, jet.load(of=lambda j, b, f=f: (_held(f(j), store), b))) for f in QU])
        st["images"] = _images(case, views, len(QU))
    elif kind == "labelled":
        jet = _Jet(dims, case["epochs"], store, seed)
        coarse, core = _boxes(dims)
        parts = []
        for box in coarse + [core]:
            size = tuple(hi - lo for lo, hi in box)
            if box is core:
                s = jet.load(tuple(2 * n for n in size), (0.5, 0.5, 0.5),
                             lambda j, b: _fine(*_cut(core, j, b)))
            else:
                s = jet.load(size, (1.0, 1.0, 1.0), lambda j, b, box=box: _cut(box, j, b))
            _lay(case, s)
            dart.dart_stack_set_placement(s, [lo for lo, _ in box], [0.5 * d for d in dims])
            parts.append(s)
        st["stack"] = dart.dart_labelled_create(parts)
        st["images"] = _images(case, views)
    elif kind == "stream":
        jet = _Jet(dims, case["epochs"], store, seed)
        fields = [jet.epoch(m) for m in range(case["epochs"])]
        st["j"] = torch.stack([f[0] for f in fields])
        st["beta"] = torch.stack([f[1] for f in fields])
        st["streamer"] = dart.dart_streamer_create(dims, (1.0, 1.0, 1.0), jet.times, STORE[store])
        st["images"] = _images(case, views)
    else:
        jet = _Jet(dims, case["epochs"], store, seed)
        st["stack"] = _lay(case, jet.load())
        st["images"] = _images(case, views)
        if kind == "frames":
            L = math.sqrt(sum(float(d) ** 2 for d in dims))
            st["frames"] = [_views(case, seed, (k - 0.5 * case["frames"]) * 0.04 * L)
                            for k in range(case["frames"])]
            st["images"] = [_images(case, views) for _ in st["frames"]]
        if kind == "refill":
            # the replaced epoch: another seed's field
            st["at"] = case["epochs"] // 2
            j, b = _Jet(dims, case["epochs"], store, seed + 1).epoch(st["at"])
            st["j"], st["beta"] = j[None].contiguous(), b[None].contiguous()
            st["back"] = (torch.empty_like(j), torch.empty_like(b))
    torch.cuda.synchronize()
    return st


def _batch(st, stack, views, images):
    """dart_render_batch on the program's side stream, in order with its own
    work on the current one."""
    s = st["stream"]
    s.wait_stream(torch.cuda.current_stream())
    flux, steps = dart.dart_render_batch([stack] * len(views), views, images, stream=s,
                                         stats=st["stats"])
    torch.cuda.current_stream().wait_stream(s)
    return {"flux": flux, "steps": steps} if st["stats"] else {}


def run(st):
    kind = st["case"]["kind"]
    if kind == "single":
        v, image = st["views"][0], st["images"][0]
        if st["stats"]:  # the image, flux and steps on the host
            host = np.empty((v.height, v.width), dtype=np.float64 if v.out_dtype == dart.DART_F64
                            else np.float32)
            flux, steps = dart.dart_render(st["stack"], v, host)
            return {"images": [host], "flux": flux, "steps": steps}
        dart.dart_render(st["stack"], v, image, stats=False)
        return {"images": [image]}
    if kind == "frames":
        for views, images in zip(st["frames"], st["images"]):
            got = _batch(st, st["stack"], views, images)
        return {"images": st["images"], **got}
    if kind == "serve":
        srv = st["server"].srv
        # the server's own streams write the images
        tickets = [dart.dart_submit(srv, s, v, im)
                   for (s, v), im in zip(st["ask"], st["images"])]
        got = [dart.dart_wait(srv, t) for t in tickets]
        return {"images": st["images"], "steps": np.array([g[1] for g in got], dtype=np.int64)}
    if kind == "stream":
        flux, steps = dart.dart_streamer_render(st["streamer"], st["j"], st["beta"], st["views"],
                                                st["images"])
        return {"images": st["images"], "flux": flux, "steps": steps}
    if kind == "refill":
        dart.dart_stack_set_epochs(st["stack"], st["at"], st["j"], st["beta"])
        got = _batch(st, st["stack"], st["views"], st["images"])
        dart.dart_stack_read_epoch(st["stack"], st["at"], *st["back"])
        return {"images": st["images"], "back": list(st["back"]), **got}
    return {"images": st["images"], **_batch(st, st["stack"], st["views"], st["images"])}


# ------------------------------------------------------------------------ work

def _shat(view):
    th, ph = math.radians(view.theta_deg), math.radians(view.phi_deg)
    n = (math.sin(th) * math.cos(ph), math.sin(th) * math.sin(ph), math.cos(th))
    return [-x if abs(x) > 1e-15 else 0.0 for x in n]


def _steps(dims, cell, view):
    """Cells the view's rays cross: (volume / pixel area) length of rays inside
    the grid times the cell faces per length."""
    vol = dims[0] * dims[1] * dims[2] * cell ** 3
    return vol / view.pixel_scale ** 2 * sum(abs(s) for s in _shat(view)) / cell


def work(case):
    """Each (cell, epoch) emissivity that the views' rays meet read once, whole
    records where matter moves (the jet's share of the volume), images written
    once; sources and records once where epochs are loaded or read back."""
    dims, kind = _dims(case), case["kind"]
    cells = dims[0] * dims[1] * dims[2]
    rec = RECORD[case["store"]]
    src = 32 if case["store"] == "f64" else 16
    views = _views(case, 0)
    moving = min(1.0, math.pi * max(2.5, 12.0 * min(dims[:2]) / 256.0) ** 2 / (dims[0] * dims[1]))
    if kind == "serve":
        # (requests fall on the stacks evenly)
        grids = [(tuple(d * g for d in dims), 1.0, min(32, case["epochs"] * e), 1.0 / len(SERVED), g)
                 for g, e in SERVED]
    elif kind == "labelled":
        coarse, core = _boxes(dims)
        size = lambda box: tuple(hi - lo for lo, hi in box)  # noqa: E731
        grids = [(size(b), 1.0, case["epochs"], 1.0, 1) for b in coarse]
        grids.append((tuple(2 * n for n in size(core)), 0.5, case["epochs"], 1.0, 1))
    else:
        grids = [(dims, 1.0, case["epochs"], 1.0, 1)]
    steps = read = 0.0
    repeat = max(1, case["frames"])
    for gdims, cell, epochs, share, scale in grids:
        n = gdims[0] * gdims[1] * gdims[2]
        seen = 0.0
        for v in views:
            s = _steps(gdims, cell, v) / scale ** 2 * share * repeat
            steps += s
            seen += 2.0 * min(s, n * share * repeat)
        chan = len(QU) if kind == "vector" else 1
        read += min(seen, float(n) * epochs) * (chan * rec / 4 + moving * rec)
    px = sum(v.width * v.height for v in views) * repeat * (8 if case["store"] == "f64" else 4)
    total = read + px * (len(QU) if kind == "vector" else 1)
    if kind == "stream":
        total = cells * case["epochs"] * src + px
    if kind == "refill":
        total += cells * (2 * src + 2 * rec)
    # per crossing: the nearest of three planes, the weight, the interpolation,
    # the chord and a compensated sum
    return {"bytes": total, "flops": 14.0 * steps * (2 if kind == "vector" else 1)}


# ----------------------------------------------------------------------- exact

CROSSINGS = 2.5e9  # plane crossings that one case's exact images may sort


def _exact_image(j, beta, times, cell, origin, centre, view):
    """The sum over cells in 64 bits: every plane crossing of a ray sorted, each
    chord at its midpoint's retarded time.  j: a list of emissivities that share
    beta; returns one image for each."""
    dev = "cuda"
    M, nz, ny, nx = j[0].shape
    n = (nx, ny, nz)
    sh = _shat(view)
    th, ph = math.radians(view.theta_deg), math.radians(view.phi_deg)
    eu = (-math.sin(ph), math.cos(ph), 0.0)
    ev = (-math.cos(th) * math.cos(ph), -math.cos(th) * math.sin(ph), math.sin(th))
    t = torch.tensor(np.asarray(times), device=dev, dtype=torch.float64)
    lookback = not view.flags & dart.DART_NO_LOOKBACK
    p = 2.0 + view.alpha
    W, H = view.width, view.height
    out = [torch.zeros(W * H, dtype=torch.float64, device=dev) for _ in j]
    flat_j = [x.reshape(-1) for x in j]
    flat_b = beta.reshape(-1, 3)
    width = sum(k + 1 for k in n) + M
    rows = max(1, int(4e7) // width)
    for r0 in range(0, W * H, rows):
        idx = torch.arange(r0, min(W * H, r0 + rows), device=dev)
        u = ((idx % W).double() + 0.5 - 0.5 * W) * view.pixel_scale
        w = ((idx // W).double() + 0.5 - 0.5 * H) * view.pixel_scale
        o = [centre[a] - origin[a] + u * eu[a] + w * ev[a] for a in range(3)]
        s_in = torch.full_like(u, -math.inf)
        s_out = torch.full_like(u, math.inf)
        for a in range(3):
            top = n[a] * cell
            if sh[a] == 0.0:
                hit = (o[a] >= 0) & (o[a] < top)
                s_out = torch.where(hit, s_out, -math.inf)
            else:
                a0, a1 = -o[a] / sh[a], (top - o[a]) / sh[a]
                s_in = torch.maximum(s_in, torch.minimum(a0, a1))
                s_out = torch.minimum(s_out, torch.maximum(a0, a1))
        keep = (s_in < s_out).nonzero()[:, 0]
        if keep.numel() == 0:
            continue
        o = [x[keep][:, None] for x in o]
        lo, hi = s_in[keep][:, None], s_out[keep][:, None]
        cuts = [lo, hi]
        for a in range(3):
            if sh[a] != 0.0:
                planes = torch.arange(n[a] + 1, device=dev, dtype=torch.float64) * cell
                cuts.append((planes[None, :] - o[a]) / sh[a])
        if view.flags & dart.DART_EXACT_TIME and lookback and M > 1:
            cuts.append((view.t_obs - t)[None, :].expand(keep.numel(), M))
        s = torch.cat(cuts, 1)
        s = torch.sort(torch.minimum(torch.maximum(s, lo), hi), 1)[0]
        ds = s[:, 1:] - s[:, :-1]
        mid = 0.5 * (s[:, 1:] + s[:, :-1])
        del s, cuts
        lin = torch.zeros(mid.shape, dtype=torch.int64, device=dev)
        for a in (2, 1, 0):
            c = torch.floor((o[a] + mid * sh[a]) / cell).long().clamp_(0, n[a] - 1)
            lin = lin * n[a] + c
        tb = view.t_obs - mid if lookback else torch.full_like(mid, view.t_obs)
        ds = torch.where((tb >= t[0]) & (tb <= t[-1]), ds, 0.0)
        m = (torch.searchsorted(t, tb, right=True) - 1).clamp_(0, max(0, M - 2))
        if M > 1:
            t0, t1 = t[m], t[(m + 1)]
            wt = (tb - t0) / (t1 - t0)
            if view.flags & dart.DART_NEAREST_EPOCH:
                wt = ((t1 - tb) < (tb - t0)).double()
        else:
            wt = torch.zeros_like(tb)
        for e in ((0, 1) if M > 1 else (0,)):
            at = (m + e) * (nx * ny * nz) + lin
            b = flat_b[at].double()
            q = 1.0 - (b * b).sum(-1)
            d = torch.sqrt(q) / (1.0 + b[..., 0] * sh[0] + b[..., 1] * sh[1] + b[..., 2] * sh[2])
            f = ds * (wt if e else 1.0 - wt) * d ** p
            for x, to in zip(flat_j, out):
                to[idx[keep]] += (f * x[at].double()).sum(1)
            del b, q, d, f, at
    return [x.reshape(H, W) for x in out]


def exact(case, seed):
    dims, kind, store = _dims(case), case["kind"], case["store"]
    left = [CROSSINGS]

    def afford(view, dd):
        cost = view.width * view.height * float(sum(dd) + 3 + case["epochs"])
        if cost > left[0]:
            return False
        left[0] -= cost
        return True

    def fields(jet, epochs, of=None):
        fs = [jet.epoch(m) if of is None else of(*jet.epoch(m)) for m in range(epochs)]
        return torch.stack([f[0] for f in fs]), torch.stack([f[1] for f in fs])

    views = _views(case, seed)
    _, stats = _options(case, 1)
    centre, zero = [0.5 * d for d in dims], (0.0, 0.0, 0.0)
    if kind == "serve":
        rng = random.Random(int(seed) + 41)
        images, held = [], {}
        for v in views:
            k = rng.randrange(len(SERVED))
            g, e = SERVED[k]
            v.pixel_scale *= g
            dd, ee = tuple(d * g for d in dims), min(32, case["epochs"] * e)
            if not afford(v, dd):
                images.append(None)
                continue
            if k not in held:
                jet = _Jet(dd, ee, store, seed + k)
                held[k] = fields(jet, ee) + (jet.times,)
            j, b, t = held[k]
            images += _exact_image([j], b, t, 1.0, zero, [0.5 * d for d in dd], v)
        return {"images": images, "steps": None}
    jet = _Jet(dims, case["epochs"], store, seed)
    if kind == "labelled":
        coarse, core = _boxes(dims)
        j, b = fields(jet, case["epochs"])
        images = []
        for v in views:
            if not afford(v, [3 * d for d in dims]):
                images.append(None)
                continue
            image = 0.0
            for box in coarse + [core]:
                cut = (slice(None),) + tuple(slice(lo, hi) for lo, hi in box[::-1])
                bj, bb, cell = j[cut], b[cut], 1.0
                if box is core:
                    for d in (1, 2, 3):
                        bj, bb = bj.repeat_interleave(2, dim=d), bb.repeat_interleave(2, dim=d)
                    cell = 0.5
                image = image + _exact_image([bj.contiguous()], bb.contiguous(), jet.times, cell,
                                             [lo for lo, _ in box], centre, v)[0]
            images.append(image)
        return {"images": images}
    j, b = fields(jet, case["epochs"])
    if kind == "refill":
        m = case["epochs"] // 2
        j[m], b[m] = _Jet(dims, case["epochs"], store, seed + 1).epoch(m)
    comps = [_held(f(j), store) for f in QU] if kind == "vector" else [j]

    def images_of(vs):
        got = []
        for v in vs:
            if not afford(v, dims):
                got.append(None)
                continue
            im = _exact_image(comps, b, jet.times, 1.0, zero, centre, v)
            got.append(torch.stack(im) if kind == "vector" else im[0])
        return got

    if kind == "frames":
        L = math.sqrt(sum(float(d) ** 2 for d in dims))
        images = [images_of(_views(case, seed, (k - 0.5 * case["frames"]) * 0.04 * L))
                  for k in range(case["frames"])]
        return {"images": images, **({"flux": None, "steps": None} if stats else {})}
    images = images_of(views)
    out = {"images": images}
    if stats or kind == "stream":
        flux = [None if im is None else float(im.sum()) * v.pixel_scale ** 2
                for im, v in zip(images, views)]
        whole = not any(f is None for f in flux)
        out["flux"] = (flux[0] if kind == "single" else np.array(flux)) if whole else None
        out["steps"] = None
    if kind == "refill":
        out["back"] = [j[m], b[m]]
    return out
