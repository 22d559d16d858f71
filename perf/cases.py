"""Timing cases of the stixel library: what a program that uses it has it do.

Each case is one call of a public entry point on device inputs that the
program already holds: one frame as it comes from the stereo stage (default
path, own camera pose, or the entry that allocates nothing), a captured batch
that is replayed, a one-call batch of uneven frames, one admission of the
serving loop, the semi-global matching stage alone, and a stereo pair taken
all the way to stixels.  Frames are ground-plus-box road scenes with noise
and invalid pixels, drawn on the device from the seed.

`listed` names the fixed cases, `draw` gives others of the same ranges,
`prepare` builds inputs and the handles a program keeps, `run` makes one
pass, `work` counts what a pass cannot do without, and `exact` evaluates the
total costs and disparity maps in plain 64-bit torch.
"""

from __future__ import annotations

import math

import torch

import paper_1610_04124_amd as stixels
from paper_1610_04124_amd import serving

INF = math.inf
GRID = 10                     # costs are multiples of 2^-10 nats

MODEL = {
    "p_out": 0.15, "sigma_disp": 1.0, "sigma_sky": 0.8, "ground_slope_noise": 0.05,
    "object_depth_extent_m": 0.3, "bic_cost": 3.0, "first_cost": [1.0, 0.0, 10.0],
    "trans_cost": [[0.5, 1.0, 0.0], [0.0, INF, 0.0], [2.0, INF, INF]],
    "ordering_cost": 4.0, "ordering_tol_px": 1, "gravity_cost": 3.0, "gravity_tol_px": 2.0,
    "diving_cost": 20.0, "diving_tol_px": 2.0,
}

#: frame sizes and stixel widths of the uneven batch
SIZES = [(640, 240, 128), (1024, 440, 128), (1280, 720, 128), (2048, 880, 256)]
WIDTHS = [3, 5, 7]

P1, P2 = 10, 120              # the matching stage's default penalties


def _case(name, kind, width, height, disparities=128, stixel_width=5, frames=1, **more):
    c = dict(kind=kind, width=width, height=height, disparities=disparities,
             stixel_width=stixel_width, frames=frames, mean=False, subpixel=0, mix=0)
    c.update(more)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest call: one small frame of one camera, waited for
        _case("frame_640x240", "frame", 640, 240),
        # the paper's headline frame, one at a time (a 30 Hz camera's latency)
        _case("frame_1024x440", "frame", 1024, 440),
        # one high-resolution frame: 256 disparities, 14 slots of rows
        _case("frame_2048x880", "frame", 2048, 880, 256),
        # a frame that brings its own horizon and pitch; a width that the
        # stixel width does not divide
        _case("pose_1280x720_s7", "pose", 1280, 720, 128, 7),
        # the entry that allocates nothing, as a loop under graph capture calls
        # it; an odd height, half-pixel disparity bins
        _case("noalloc_1024x437_half_px", "noalloc", 1024, 437, 128, 5, subpixel=1),
        # one admission of the serving loop: frames of two cameras that wait
        # together, outputs allocated, a launch per height class, polled
        _case("serve_3_frames", "serve", 1024, 440, 128, 5, 3),
        # the headline batch: 64 frames, captured once and replayed
        _case("batch64_1024x440", "batch", 1024, 440, 128, 5, 64),
        # high-resolution batch with narrow stixels, the paper's mean reduction
        _case("batch16_2048x880_s3_mean", "batch", 2048, 880, 256, 3, 16, mean=True),
        # cameras of four sizes and three stixel widths in one call
        _case("uneven_64_frames", "uneven", 2048, 880, 256, 5, 64, mix=1),
        # the matching stage: one pair as it arrives, and an offline batch
        _case("sgm_1024x440", "sgm", 1024, 440),
        _case("sgm_64x1024x440", "sgm", 1024, 440, frames=64),
        # pair in, stixels out: ragged small images, 64 disparities
        _case("stereo_641x241_d64", "stereo", 641, 241, 64),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["frame", "frame", "pose", "noalloc", "batch", "batch", "uneven", "serve",
                       "sgm", "sgm", "stereo"])
    w, h = _log_int(rng, 320, 2048), _log_int(rng, 120, 960)
    if kind in ("sgm", "stereo"):
        w, h = _log_int(rng, 320, 1600), _log_int(rng, 120, 800)
        d = rng.choice([32, 64, 96, 128, 192, 256])
        n = 1
        if kind == "sgm":
            n = _log_int(rng, 1, 32)
            n = max(1, min(n, 2_500_000_000 // (w * h * d)))
        return _case("", kind, w, h, d, rng.choice(WIDTHS), n)
    d = rng.choice([64, 128, 128, 200, 256])
    s = rng.choice([2, 3, 5, 5, 7, 9])
    sub = 1 if kind == "noalloc" and d <= 128 and rng.random() < 0.5 else 0
    n = 1
    if kind == "serve":
        n = rng.randint(1, 6)
        d = 128
        h = min(h, 500)
    if kind == "batch":
        n = _log_int(rng, 2, 64)
        n = max(2, min(n, 2_000_000_000 // ((w // s) * h * h // 2)))
    if kind == "uneven":
        n = _log_int(rng, 4, 48)
        w, h, d = SIZES[-1]
    return _case("", kind, w, h, d, s, n, mean=rng.random() < 0.25, subpixel=sub,
                 mix=rng.randint(2, 10_000) if kind == "uneven" else 0)


# ------------------------------------------------------------------ inputs
def _camera(width, height):
    return {"focal_px": 700.0 * width / 1024.0, "baseline_m": 0.3, "cam_height_m": 1.2,
            "horizon_row": float(round(180.0 * height / 440.0)), "pitch_rad": 0.0}


def _params(width, height, disparities, s, mean=False, subpixel=0, batch_only=False):
    return {"camera": _camera(width, height), "model": MODEL, "stixel_width": s,
            "max_disparity": disparities, "max_width": width, "max_height": height,
            "max_stixels_per_column": 0, "reduce_mode": 1 if mean else 0,
            "cost_grid_log2": GRID, "flags": 1 if batch_only else 0, "subpixel_log2": subpixel}


def _pose(height):
    return (float(round(180.0 * height / 440.0)) + 5.5, 0.02)


def _groups(case):
    """The frames of a case as groups of one size: (width, height, disparities, s, count)."""
    n, k = case["frames"], case["kind"]
    if k == "uneven":
        mix, count = case["mix"] * 2654435761 % 2**32, {}
        for _ in range(n):
            mix = (mix * 1103515245 + 12345) % 2**31
            w, h, d = SIZES[(mix >> 16) % 4]
            key = (w, h, d, WIDTHS[(mix >> 20) % 3])
            count[key] = count.get(key, 0) + 1
        return [(*key, c) for key, c in sorted(count.items())]
    one = (case["width"], case["height"], case["disparities"], case["stixel_width"])
    if k == "serve" and n > 1:
        # two cameras: one frame in three from a taller one
        return [(*one, n - n // 3), (1280, 720, 128, case["stixel_width"], n // 3)] if n >= 3 \
            else [(*one, n)]
    return [(*one, n)]


def _scene(width, height, d_max, n, gen):
    """Noise-free disparity [n, H, W] and sky mask of n road scenes."""
    dev = gen.device
    cam = _camera(width, height)
    f, base, hc, hr = cam["focal_px"], cam["baseline_m"], cam["cam_height_m"], cam["horizon_row"]

    def uni(lo, hi, *shape):
        return lo + (hi - lo) * torch.rand(shape, generator=gen, device=dev)

    rows = torch.arange(height, device=dev, dtype=torch.float32)[None, :, None]
    cols = torch.arange(width, device=dev, dtype=torch.float32)[None, None, :]
    disp = torch.where(rows > hr, (base / hc) * (rows - hr), torch.zeros_like(rows))
    disp = disp.expand(n, height, width).contiguous()
    sky = (rows <= hr).expand(n, height, width).clone()
    boxes = 4 + (9 * torch.rand(n, generator=gen, device=dev)).long()
    z, tall, wide, at = (uni(5.0, 60.0, 12, n), uni(0.5, 3.0, 12, n),
                         uni(16.0, 160.0, 12, n) * width / 1024.0, uni(0.0, 1.0, 12, n))
    for i in range(12):
        d = f * base / z[i]
        foot = hr + f * hc / z[i]
        top = foot - f * tall[i] / z[i]
        left = at[i] * (width - wide[i]).clamp(min=0.0)
        v = lambda x: x[:, None, None]  # noqa: E731
        m = ((rows >= v(top)) & (rows <= v(foot)) & (cols >= v(left)) & (cols < v(left + wide[i]))
             & (v(d) >= disp) & v(boxes > i))
        disp = torch.where(m, v(d).expand_as(disp), disp)
        sky &= ~m
    return disp.clamp_(max=d_max - 1.0), sky


def _frames(width, height, d_max, n, gen):
    disp, _ = _scene(width, height, d_max, n, gen)
    disp += 0.8 * torch.randn(disp.shape, generator=gen, device=gen.device)
    disp.clamp_(0.0, d_max - 1.0)
    disp[torch.rand(disp.shape, generator=gen, device=gen.device) < 0.05] = -1.0
    return disp


def _pairs(width, height, d_max, n, gen):
    """n rectified pairs (uint8): the right view is the left one warped by the
    scene's whole-pixel disparity, nearest surface in front."""
    dev = gen.device
    disp, sky = _scene(width, height, d_max, n, gen)
    d = disp.round().long()

    def texture(lo, hi):
        t = lo + (hi - lo) * torch.rand((n, height + 1, width + 1), generator=gen, device=dev)
        return 0.25 * (t[:, :-1, :-1] + t[:, 1:, :-1] + t[:, :-1, 1:] + t[:, 1:, 1:])

    left = torch.where(sky, 128.0 + texture(-24.0, 24.0), texture(20.0, 235.0))
    x = torch.arange(width, device=dev)[None, None, :] - d
    key = torch.where(x >= 0, d * 65536 + (left * 128.0).long(), torch.full_like(d, -1))
    seen = torch.full_like(d, -1).scatter_reduce_(2, x.clamp(min=0), key, "amax")
    right = torch.where(seen >= 0, (seen % 65536).float() / 128.0, texture(20.0, 235.0))

    def image(t):
        t = t + torch.randn(t.shape, generator=gen, device=dev)
        return t.round().clamp(0, 255).to(torch.uint8)

    return image(left), image(right)


def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _inputs(case, seed):
    """Input tensors of each group of a case."""
    gen, got = _generator(seed), []
    for w, h, d, _, n in _groups(case):
        got.append(_pairs(w, h, d, n, gen) if case["kind"] in ("sgm", "stereo")
                   else _frames(w, h, d, n, gen))
    return got


# ------------------------------------------------------------------ a pass
def prepare(case, seed):
    kind, groups, inputs = case["kind"], _groups(case), _inputs(case, seed)
    st = {"kind": kind, "inputs": inputs}
    w, h, d, s, n = groups[0]
    if kind in ("sgm", "stereo"):
        left, right = inputs[0]
        st["sgm"] = stixels.Sgm(w, h, d, max_frames=n)
        if kind == "stereo":
            st["pair"] = (left[0].contiguous(), right[0].contiguous())
            st["handle"] = stixels.Stixels(_params(w, h, d, s))
            st["out"] = st["handle"].new_output(w, h)
        else:
            st["pair"] = (left, right)
        st["map"] = torch.empty(st["pair"][0].shape, dtype=torch.float32, device="cuda")
        return st
    handles = [stixels.Stixels(_params(gw, gh, gd, gs, case["mean"], case["subpixel"],
                                       kind in ("batch", "uneven", "serve")))
               for gw, gh, gd, gs, _ in groups]
    if kind in ("frame", "pose", "noalloc"):
        st["handle"], st["frame"] = handles[0], inputs[0][0].contiguous()
        st["out"] = handles[0].new_output(w, h)
        st["pose"] = _pose(h) if kind == "pose" else None
        return st
    if kind == "serve":
        cameras = [serving.CameraSpec(hd, gw, gh) for hd, (gw, gh, *_) in zip(handles, groups)]
        st["executor"] = serving.GpuExecutor(cameras, max_frames=8)
        st["frames"] = [(i, f) for i, fs in enumerate(inputs) for f in fs.unbind(0)]
        return st
    st["items"], st["outputs"] = [], []
    for hd, (gw, gh, *_), fs in zip(handles, groups, inputs):
        outs, stacked = _stacked(hd, gw, gh, len(fs))
        st["items"] += [(hd, f, o) for f, o in zip(fs.unbind(0), outs)]
        st["outputs"].append(stacked)
    if kind == "batch":
        # the launch layout the serving loop uses for this height
        st["stream"] = torch.cuda.Stream()
        st["stream"].wait_stream(torch.cuda.current_stream())
        st["batch"] = stixels.Batch(n, n * (w // s), h, d)
        st["batch"].set_waves(1 if h <= 512 else 2)
        st["batch"].capture(st["items"], st["stream"])
    return st


def _stacked(handle, width, height, n):
    """Outputs of n frames of one size as slices of four stacked tensors, and those tensors."""
    outs = [handle.new_output(width, height) for _ in range(n)]
    whole = {k: torch.stack([getattr(o, k) for o in outs])
             for k in ("counts", "records", "total", "overflow")}
    for k, t in whole.items():
        for o, x in zip(outs, t.unbind(0)):
            setattr(o, k, x)
    return outs, whole


def _outputs(o):
    return {"counts": o.counts, "records": o.records, "total": o.total, "overflow": o.overflow}


def run(state):
    kind = state["kind"]
    if kind == "sgm":
        return {"disparity": state["sgm"].compute(*state["pair"], state["map"])}
    if kind == "stereo":
        out, disparity = state["handle"].compute_stereo(state["sgm"], *state["pair"], state["out"],
                                                        state["map"])
        return dict(_outputs(out), disparity=disparity)
    if kind in ("frame", "pose"):
        return _outputs(state["handle"].compute(state["frame"], state["out"], pose=state["pose"]))
    if kind == "noalloc":
        return _outputs(state["handle"].compute_noalloc(state["frame"], state["out"]))
    if kind == "serve":
        reqs = [serving.Request(i, c, f, 0.0) for i, (c, f) in enumerate(state["frames"])]
        token = state["executor"].launch(reqs)
        while not state["executor"].finished(token):
            pass
        return [_outputs(r.out) for r in reqs]
    if kind == "uneven":
        stixels.compute_batch(state["items"])
    else:
        state["batch"].replay(state["stream"])
    return state["outputs"]


def work(case):
    """Inputs read once and outputs written once; 13 operations for each (cut,
    row) pair of the recurrence, 10 for each (pixel, disparity, path)."""
    nbytes = flops = 0.0
    for w, h, d, s, n in _groups(case):
        if case["kind"] in ("sgm", "stereo"):
            nbytes += n * w * h * (2 + 4)
            flops += 40.0 * n * w * h * d
        if case["kind"] != "sgm":
            cols = w // s
            # counts, total, overflow and about eight records a column
            nbytes += n * (4.0 * w * h + cols * (9 + 8 * 12))
            flops += 13.0 * n * cols * h * (h + 1) / 2
    return {"bytes": nbytes, "flops": flops}


# ------------------------------------------------------------------ in 64 bits
def _grid(x):
    return torch.round(x * 2.0**GRID) * 2.0**-GRID


def _pixel_cost(d, mu, sigma, d_range):
    """Outlier cost or Gaussian cost, whichever is smaller, of disparity d under a model mean mu."""
    p = MODEL["p_out"]
    cdf = lambda x: 0.5 * torch.special.erfc(-x / math.sqrt(2.0))  # noqa: E731
    out = math.log(d_range) - math.log(p)
    mass = cdf((d_range - mu) / sigma) - cdf(-mu / sigma)
    g = (torch.log(mass) + torch.log(sigma * math.sqrt(2.0 * math.pi)) - math.log(1.0 - p)
         + (d - mu) ** 2 / (2.0 * sigma * sigma))
    return _grid(torch.where(torch.isfinite(g) & (g < out), g, torch.full_like(g, out)))


def _reduced(frames, s, bins, mean, sub):
    """Bottom-up reduced pixels [n * ncols, H], -1 invalid."""
    n, h, w = frames.shape
    x = frames[:, :, :w // s * s].reshape(n, h, w // s, s).double()
    ok = torch.isfinite(x) & (x >= 0)
    count = ok.sum(-1)
    if mean:
        m = torch.where(ok, x, torch.zeros_like(x)).sum(-1) / count.clamp(min=1)
    else:
        srt = torch.where(ok, x, torch.full_like(x, INF)).sort(-1).values
        m = srt.gather(-1, ((count - 1).clamp(min=0) // 2)[..., None])[..., 0]
    q = torch.where(count > 0, torch.round(m * 2.0**sub).clamp(max=bins - 1.0),
                    torch.full_like(m, -1.0))
    return q.long().flip(1).permute(0, 2, 1).reshape(n * (w // s), h)


def _totals(frames, w, h, disparities, s, mean=False, sub=0, pose=None):
    """Total cost of every column, [n, ncols]."""
    dev = frames.device
    cam = _camera(w, h)
    if pose is not None:
        cam["horizon_row"], cam["pitch_rad"] = pose
    bins, dr = disparities << sub, float(disparities)
    q_all = _reduced(frames, s, bins, mean, sub)
    f64 = dict(dtype=torch.float64, device=dev)
    px = torch.arange(bins, **f64) * 2.0**-sub
    v = torch.arange(h + 1, **f64)
    alpha = cam["baseline_m"] * math.cos(cam["pitch_rad"]) / cam["cam_height_m"]
    vhor = (h - 1) - cam["horizon_row"]
    vtop = max(-1, min(h, math.floor(vhor)))
    ground = alpha * (vhor - v)
    sky = _pixel_cost(px, torch.zeros((), **f64), torch.tensor(MODEL["sigma_sky"], **f64), dr)
    sg = torch.sqrt(1.0 + (MODEL["ground_slope_noise"] * ground) ** 2)
    gtab = _pixel_cost(px[None, :], ground[:h, None], sg[:h, None], dr)
    gtab[vtop + 1:] = 0.0
    so = torch.sqrt(1.0 + (px * px * MODEL["object_depth_extent_m"]
                           / (cam["focal_px"] * cam["baseline_m"])) ** 2)
    otab = _pixel_cost(px[:, None], px[None, :], so[None, :], dr)       # [pixel][mean]
    hi = torch.floor((ground + MODEL["diving_tol_px"]) * 2.0**sub)
    lo = torch.ceil((ground - MODEL["gravity_tol_px"]) * 2.0**sub)
    beta, tau = MODEL["bic_cost"], MODEL["ordering_tol_px"] << sub
    first = [c + beta for c in MODEL["first_cost"]]
    tr = [[c + beta for c in row] for row in MODEL["trans_cost"]]
    got = []
    for q in q_all.split(max(1, 500_000_000 // (bins * (h + 1)))):
        n = q.shape[0]
        ok, qc = q >= 0, q.clamp(min=0)

        def prefix(x):
            out = torch.zeros((n, h + 1), dtype=x.dtype, device=dev)
            out[:, 1:] = torch.where(ok, x, torch.zeros_like(x)).cumsum(1)
            return out

        pg = prefix(gtab[torch.arange(h, device=dev)[None, :], qc])
        ps, pd, pn = prefix(sky[qc]), prefix(qc), prefix(torch.ones_like(qc))
        po = torch.zeros((n, h + 1, bins), **f64)
        po[:, 1:] = torch.where(ok[..., None], otab[qc], torch.zeros((), **f64)).cumsum(1)

        def mean_of(b):
            cnt, tot = pn[:, b + 1:] - pn[:, b:b + 1], pd[:, b + 1:] - pd[:, b:b + 1]
            return torch.div(2 * tot + cnt, (2 * cnt).clamp(min=1), rounding_mode="floor")

        f = mean_of(0)
        ob = po[:, 1:].gather(2, f[..., None])[..., 0] + first[0]
        fob = f
        rg, rs = (torch.full((n,), first[c], **f64) for c in (1, 2))
        inf = torch.full((n,), INF, **f64)
        for j in range(h):
            co, cs = ob[:, j], ps[:, j + 1] + rs
            cg = pg[:, j + 1] + rg if j <= vtop else inf
            b = j + 1
            if b == h:
                got.append(torch.minimum(torch.minimum(co, cg), cs))
                break
            xs = torch.minimum(torch.minimum(co + tr[0][2], cg + tr[1][2]), cs + tr[2][2])
            rs = torch.minimum(rs, xs - ps[:, b])
            if b <= vtop:
                xg = torch.minimum(torch.minimum(co + tr[0][1], cg + tr[1][1]), cs + tr[2][1])
                rg = torch.minimum(rg, xg - pg[:, b])
            f = mean_of(b)
            data = (po[:, b + 1:].gather(2, f[..., None])[..., 0]
                    - po[:, b].gather(1, f))
            pen = MODEL["ordering_cost"] * (f > fob[:, j:j + 1] + tau)
            x = co[:, None] + tr[0][0] + pen
            if j <= vtop:
                pen = torch.where(f > hi[b], MODEL["diving_cost"],
                                  torch.where(f < lo[b], MODEL["gravity_cost"], 0.0))
                x = torch.minimum(x, cg[:, None] + tr[1][0] + pen)
            x = torch.minimum(x, cs[:, None] + tr[2][0]) + data
            better = x < ob[:, b:]
            ob[:, b:] = torch.where(better, x, ob[:, b:])
            fob = torch.cat([fob[:, :b], torch.where(better, f, fob[:, b:])], 1)
        del po
    return torch.cat(got).reshape(frames.shape[0], w // s)


def _census(img):
    """62 comparison bits of every pixel, [n, H, W] words."""
    n, h, w = img.shape
    pad = torch.full((n, h + 6, w + 8), 256, dtype=torch.int64, device=img.device)
    pad[:, 3:-3, 4:-4] = img
    word, bit = torch.zeros((n, h, w), dtype=torch.int64, device=img.device), 0
    for dy in range(7):
        for dx in range(9):
            if (dy, dx) != (3, 4):
                word |= (pad[:, dy:dy + h, dx:dx + w] < img).long() << bit
                bit += 1
    return word


def _popcount(x):
    x = x - ((x >> 1) & 0x5555555555555555)
    x = (x & 0x3333333333333333) + ((x >> 2) & 0x3333333333333333)
    x = (x + (x >> 4)) & 0x0F0F0F0F0F0F0F0F
    return ((x * 0x0101010101010101) >> 56) & 0xFF


def _disparity(left, right, d_max):
    """Semi-global matching with four paths, in whole numbers: [n, H, W] float64."""
    n, h, w = left.shape
    cl, cr = _census(left.long()), _census(right.long())
    x = torch.arange(w, device=left.device)
    cost = torch.full((n, h, w, d_max), 62, dtype=torch.int32, device=left.device)
    for d in range(min(d_max, w)):
        cost[:, :, d:, d] = _popcount(cl[:, :, d:] ^ cr[:, :, :w - d]).int()
    total = torch.zeros_like(cost)
    big = 1 << 20
    for axis, back in ((1, False), (1, True), (2, False), (2, True)):
        prev = None
        steps = range(cost.shape[axis])
        for i in reversed(steps) if back else steps:
            c = cost.select(axis, i)
            if prev is None:
                cur = c.clone()
            else:
                m = prev.amin(-1, keepdim=True)
                edge = torch.full_like(m, big)
                nb = torch.minimum(torch.cat([edge, prev[..., :-1]], -1),
                                   torch.cat([prev[..., 1:], edge], -1)) + P1
                cur = c + torch.minimum(torch.minimum(prev, nb), m + P2) - m
            total.select(axis, i).add_(cur)
            prev = cur
    del cost
    dl = (total == total.amin(-1, keepdim=True)).int().argmax(-1)   # the smallest disparity
    best = torch.full((n, h, w), 1 << 30, dtype=torch.int32, device=left.device)
    for d in range(min(d_max, w)):
        best[:, :, :w - d] = torch.minimum(best[:, :, :w - d], total[:, :, d:, d] * 256 + d)
    xr = x[None, None, :] - dl
    dr = (best % 256).long().gather(2, xr.clamp(min=0))
    good = (xr >= 0) & ((dl - dr).abs() <= 1)
    return torch.where(good, dl.double(), torch.full_like(dl, -1, dtype=torch.float64))


def exact(case, seed):
    kind, groups, inputs = case["kind"], _groups(case), _inputs(case, seed)

    def outputs(total):
        return {"counts": None, "records": None, "total": total, "overflow": None}

    w, h, d, s, n = groups[0]
    if kind in ("sgm", "stereo"):
        left, right = inputs[0]
        step = max(1, 1_000_000_000 // (w * h * d))
        maps = torch.cat([_disparity(a, b, d) for a, b in zip(left.split(step), right.split(step))])
        if kind == "sgm":
            return {"disparity": maps}
        return dict(outputs(_totals(maps, w, h, d, s)[0]), disparity=maps[0])
    got = []
    for (gw, gh, gd, gs, _), frames in zip(groups, inputs):
        pose = _pose(gh) if kind == "pose" else None
        totals = _totals(frames, gw, gh, gd, gs, case["mean"], case["subpixel"], pose)
        got += [outputs(totals)] if kind in ("batch", "uneven") else [outputs(t) for t in totals]
    return got[0] if kind in ("frame", "pose", "noalloc") else got
