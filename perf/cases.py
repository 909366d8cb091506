"""The work a user of this framework has it do, as measurable cases.

Every case is one pass through public entry points of `fastgrid` on data that
is already in device memory, as a camera pipeline keeps it:

  detect    one frame through Context.detect (pyramid, scores, NMS, cells)
  plan      a resident batch of frames, one Context.plan_launch
  submit    a batch of frames of a serving loop, one Context.submit with at
            most four submissions in flight
  maps      Context.score_maps, then Context.nms_grid on the maps
  pyramid   Context.pyr_build
  track     Context.track of a feature list, from zero estimates
  frontend  one step of the detect-and-track loop of several cameras: a
            batched SAD-A detection, then fast_frontend_step

Sizes, levels, thresholds, arc lengths and cells are those of the package's
synthetic workloads (`synth`) and of the tests; tracking stops at a step small
enough that any two correct trackers agree closely; frames are the package's
shape scenes with fresh Gaussian noise, or, where features are tracked,
textured scenes under a known motion.
"""
from __future__ import annotations

import collections
import math
import random
from types import SimpleNamespace

import torch

from paper_2003_13493_amd import fastgrid, synth

THRESHOLDS = (8, 10, 15, 20)
ARCS = (9, 10, 12)
CELLS = (16, 32, 64)
SCORES = {"sadb": fastgrid.FAST_SCORE_SADB, "sada": fastgrid.FAST_SCORE_SADA, "mt": fastgrid.FAST_SCORE_MT}
MODE = fastgrid.FAST_TRACK_GAIN | fastgrid.FAST_TRACK_OFFSET
MAX_ITER = 30


def listed():
    return [
        # the smallest call: one low-resolution frame, one level, where the launch is most of the time
        _detect("detect-320x240", 320, 240, 1, 10, 9, 32, "sadb"),
        # one frame of a VGA-class camera (EuRoC's size), three levels
        _detect("detect-752x480", 752, 480, 3, 10, 10, 32, "sadb"),
        # one full-HD frame, four levels, coarse cells
        _detect("detect-1920x1080", 1920, 1080, 4, 15, 9, 64, "sadb"),
        # the largest camera frame, five levels, with the arc score of the tracking front end
        _detect("detect-4096x2160", 4096, 2160, 5, 10, 10, 32, "sada"),
        # the throughput workload: 64 resident frames of three sizes in one launch
        {"name": "plan-64-frames", "kind": "plan", "sizes": "752x480*24,1280x720*24,640x480*16", "levels": "3",
         "mix": 4},
        # a serving batch of mixed cameras, three to five levels, an odd size among them
        {"name": "submit-8-cameras", "kind": "submit",
         "sizes": "640x480*2,752x480*2,1920x1080*2,4096x2160,1283x719", "levels": "3,4,5", "mix": 5},
        # separate score maps and NMS, at a size that no tile divides
        {"name": "maps-641x479", "kind": "maps", "width": 641, "height": 479, "levels": 3, "t": 10, "n": 9, "cell": 16,
         "score": "sadb", "radius": 1},
        # the same on full HD with the maximum-threshold score and the widest window
        {"name": "maps-1920x1080", "kind": "maps", "width": 1920, "height": 1080, "levels": 4, "t": 15, "n": 9,
         "cell": 32, "score": "mt", "radius": 4},
        # the pyramid alone, as the one-camera front end builds it before tracking
        {"name": "pyramid-1920x1080", "kind": "pyramid", "width": 1920, "height": 1080, "levels": 4},
        # the paper's tracking workload: 100 features of one camera
        {"name": "track-100", "kind": "track", "width": 752, "height": 480, "levels": 3, "features": 100,
         "eps": 0.0001},
        # many features on a large frame: throughput of the tracker
        {"name": "track-10000", "kind": "track", "width": 1920, "height": 1080, "levels": 3, "features": 10000,
         "eps": 0.0001},
        # one step of sixteen cameras with 100 tracks each, re-detection at the paper's 30%
        {"name": "frontend-16-cameras", "kind": "frontend", "width": 752, "height": 480, "levels": 3, "t": 10, "n": 9,
         "cell": 32, "cameras": 16, "target": 100, "below": 0.3, "eps": 0.0001},
    ]


def _detect(name, w, h, levels, t, n, cell, score):
    return {"name": name, "kind": "detect", "width": w, "height": h, "levels": levels, "t": t, "n": n, "cell": cell,
            "score": score}


def draw(rng):
    """One more case of the same ranges; sizes log-uniform, of any parity."""
    kind = rng.choice(("detect", "detect", "plan", "submit", "maps", "maps", "pyramid", "track", "track", "frontend"))
    w, h = _draw_size(rng, 160, 4096)
    levels = rng.randint(1, 5)
    p = {"t": rng.choice(THRESHOLDS), "n": rng.choice(ARCS), "cell": rng.choice(CELLS)}
    score = rng.choice(("sadb", "sadb", "sada", "mt"))
    if kind == "detect":
        return {"kind": kind, "width": w, "height": h, "levels": levels, **p, "score": score}
    if kind in ("plan", "submit"):
        most = 64 if kind == "plan" else 12
        frames, sizes = int(round(math.exp(rng.uniform(math.log(2), math.log(most))))), []
        budget = 30e6 if kind == "plan" else 14e6
        for _ in range(frames):
            fw, fh = _draw_size(rng, 320, 1920 if kind == "plan" else 4096)
            if sum(a * b for a, b in sizes) + fw * fh <= budget or not sizes:
                sizes.append((fw, fh))
        return {"kind": kind, "sizes": ",".join("%dx%d" % s for s in sizes),
                "levels": "3" if kind == "plan" else "3,4,5", "mix": rng.randint(10, 10 ** 6)}
    if kind == "maps":
        w, h = _draw_size(rng, 160, 1920)
        return {"kind": kind, "width": w, "height": h, "levels": levels, **p, "score": score,
                "radius": rng.randint(1, 4)}
    if kind == "pyramid":
        return {"kind": kind, "width": w, "height": h, "levels": rng.randint(2, 6)}
    if kind == "track":
        w, h = _draw_size(rng, 640, 1920)
        return {"kind": kind, "width": w, "height": h, "levels": rng.randint(1, 3),
                "features": int(round(math.exp(rng.uniform(math.log(30), math.log(10000))))), "eps": 0.0001}
    w, h = _draw_size(rng, 320, 1280)
    return {"kind": kind, "width": w, "height": h, "levels": rng.randint(2, 3), **p, "cameras": rng.randint(1, 16),
            "target": rng.choice((50, 100, 150, 300)), "below": rng.choice((0.3, 0.3, 0.95)), "eps": 0.0001}


def _draw_size(rng, lo, hi):
    w = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    return w, max(120, int(round(w * rng.uniform(0.5, 0.8))))


# ------------------------------------------------------------------ inputs

_ctx = None
_in_flight = collections.deque()   # tickets of submissions whose job tables are in use


def _context():
    """The program's one context (with the shipped launch-shape table)."""
    global _ctx
    if _ctx is None:
        _ctx = fastgrid.Context(0)
    return _ctx


def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _noisy(img, gen, sigma):
    """A uint8 frame of the float image plus Gaussian noise."""
    noise = torch.randn(img.shape, generator=gen, device="cuda", dtype=torch.float32)
    return (img.float() + sigma * noise + 0.5).floor().clamp(0, 255).to(torch.uint8)


def _shapes(w, h, seed, gen, sigma=4.0):
    """A shape scene of the package with fresh noise."""
    count = 60 if w * h < 100_000 else 120 if w * h < 1_000_000 else 400
    return _noisy(torch.from_numpy(synth.scene(w, h, seed, count)).cuda(), gen, sigma)


def _waves(w, h, levels, rng, dx=0.0, dy=0.0):
    """A smooth field of plane waves moved by (dx, dy), float64 around 0; the
    waves are long enough for the coarsest level to resolve them and short
    enough to give the finest texture, so that every track has one answer."""
    shortest, longest = max(14.0, 2.4 * 2 ** (levels - 1)), max(42.0, 8.0 * 2 ** (levels - 1))
    y = torch.arange(h, device="cuda", dtype=torch.float64)[:, None] - dy
    x = torch.arange(w, device="cuda", dtype=torch.float64)[None, :] - dx
    f = torch.zeros((h, w), device="cuda", dtype=torch.float64)
    for _ in range(8):
        wl, th, ph = rng.uniform(shortest, longest), rng.uniform(0.0, math.pi), rng.uniform(0.0, 2.0 * math.pi)
        f += rng.uniform(7.0, 12.0) * torch.sin(2.0 * math.pi / wl * (math.cos(th) * x + math.sin(th) * y) + ph)
    return f


class _Frames:
    """Pyramids and cell slots of several frames, resident in two device
    buffers (level planes past the input, and slots), with the inputs apart."""

    def __init__(self, shapes):
        dims = [fastgrid.fast_pyr_dims(w, h, levels) for w, h, levels, _ in shapes]
        grids = [fastgrid.fast_grid_dims(w, h, cell) for w, h, _, cell in shapes]
        sizes = [[p * h for _, h, p in d[1:]] for d in dims]
        self.upper = torch.zeros(max(1, sum(map(sum, sizes))), dtype=torch.uint8, device="cuda")
        self.slots = torch.zeros(sum(a * b * 8 for a, b in grids), dtype=torch.uint8, device="cuda")
        self.inputs, self.pyr, self.grid = [], [], []
        at, slot = self.upper.data_ptr(), self.slots.data_ptr()
        for (w, h, levels, _), d, g in zip(shapes, dims, grids):
            img = torch.zeros((h, d[0][2]), dtype=torch.uint8, device="cuda")
            self.inputs.append(img)
            planes = (fastgrid.fast_plane * levels)()
            planes[0] = fastgrid.fast_plane(img.data_ptr(), w, h, d[0][2])
            for k in range(1, levels):
                planes[k] = fastgrid.fast_plane(at, *d[k])
                at += d[k][1] * d[k][2]
            self.pyr.append(SimpleNamespace(planes=planes, levels=levels, width=w, height=h))
            self.grid.append(SimpleNamespace(ptr=slot))
            slot += g[0] * g[1] * 8

    def fill(self, i, img):
        self.inputs[i][:, :img.shape[1]].copy_(img)

    def outputs(self):
        return [self.slots, self.upper]


def _mix(case):
    """The frames of a batch: (w, h, levels, t, n, cell, score), in a seeded order."""
    rng, sizes = random.Random(case["mix"]), []
    for part in case["sizes"].split(","):
        size, _, times = part.partition("*")
        sizes += [tuple(map(int, size.split("x")))] * int(times or 1)
    rng.shuffle(sizes)
    levels = [int(v) for v in case["levels"].split(",")]
    return [(w, h, rng.choice(levels), rng.choice(THRESHOLDS), rng.choice(ARCS), rng.choice(CELLS), "sadb")
            for w, h in sizes]


def _motion(seed):
    rng = random.Random(seed * 31 + 7)
    return rng.uniform(-4.0, 4.0), rng.uniform(-4.0, 4.0)


CANDIDATES = 8


def _features(img, levels, count, rng, margin):
    """`count` features of a frame, one in each cell of a grid inside a
    margin: of a few positions the one whose patches fix their motion best,
    as a detector picks corners."""
    h, w = img.shape
    cols = max(1, int(round(math.sqrt(count * (w - 2 * margin) / max(1, h - 2 * margin)))))
    rows = -(-count // cols)
    at = [(margin + (i % cols + rng.random()) * (w - 2 * margin) / cols,
           margin + (i // cols + rng.random()) * (h - 2 * margin) / rows)
          for i in range(count) for _ in range(CANDIDATES)]
    at = torch.tensor(at, dtype=torch.float32).cuda()
    worst = torch.full((len(at),), math.inf, dtype=torch.float64, device="cuda")
    for k, level in enumerate(_pyramid64(img, levels)):
        p, half = at.double() / (1 << k), 8 if k < 2 else 4
        fits = _inside(p, level, -half - 1, half)
        u = _steepest(level, p[fits], half, torch.ones((1, 1), dtype=torch.float64, device="cuda"))
        u = u / (u * u).sum(1, keepdim=True).sqrt().clamp(min=1e-9)
        det = torch.diagonal(_cholesky(u)[0], dim1=1, dim2=2).prod(1)   # 1: four independent parameters
        worst[fits] = torch.minimum(worst[fits], det)
    best = worst.reshape(count, CANDIDATES).argmax(1)
    return at.reshape(count, CANDIDATES, 2)[torch.arange(count, device="cuda"), best].contiguous()


def _track_inputs(case, seed):
    """Two frames of a textured scene under a sub-pixel motion and a change of
    light, and the features of the first."""
    w, h = case["width"], case["height"]
    rng, gen, (dx, dy) = random.Random(seed), _generator(seed), _motion(seed)
    waves = rng.getrandbits(32)
    frames = [_noisy(gain * (128.0 + _waves(w, h, case["levels"], random.Random(waves), x, y)) + light, gen, 1.0)
              for x, y, gain, light in ((0.0, 0.0, 1.0, 0.0), (dx, dy, 1.06, -5.0))]
    return frames, _features(frames[0], case["levels"], case["features"], rng, 24)


def _camera_inputs(case, seed, camera):
    """Two crops of a scene of shapes and texture, moved by whole pixels, and
    the features that live in the first."""
    w, h = case["width"], case["height"]
    seed = seed * 64 + camera
    rng, gen = random.Random(seed), _generator(seed)
    shapes = torch.from_numpy(synth.scene(w + 16, h + 16, seed, 120)).cuda().double()
    scene = (0.3 * shapes + _waves(w + 16, h + 16, case["levels"], rng) + 90.0).clamp(0, 255)
    frames = []
    for ox, oy in ((8, 8), (8 + rng.randint(-3, 3), 8 + rng.randint(-3, 3))):
        frames.append(_noisy(scene[oy:oy + h, ox:ox + w], gen, 1.0))
    return frames, _features(frames[0], case["levels"], case["target"], rng, 24)


def prepare(case, seed):
    kind, ctx, gen = case["kind"], _context(), _generator(seed)
    s = SimpleNamespace(kind=kind, case=case, ctx=ctx)
    if kind in ("detect", "maps", "pyramid"):
        w, h, levels = case["width"], case["height"], case["levels"]
        s.pyr = fastgrid.Pyramid(w, h, levels)
        s.pyr.tensors[0][:, :w].copy_(_shapes(w, h, seed, gen))
        if kind != "pyramid":
            s.grid = fastgrid.Grid(w, h, case["cell"])
            s.score = SCORES[case["score"]]
        if kind == "maps":
            s.maps = fastgrid.ScoreMaps(w, h, levels)
    elif kind in ("plan", "submit"):
        mix = _mix(case)
        s.frames = _Frames([(w, h, levels, cell) for w, h, levels, _, _, cell, _ in mix])
        for i, f in enumerate(mix):
            s.frames.fill(i, _shapes(f[0], f[1], seed * 100 + i, gen))
        s.jobs = ctx.make_jobs((p, t, n, cell, g, SCORES[score]) for (_, _, _, t, n, cell, score), p, g
                               in zip(mix, s.frames.pyr, s.frames.grid))
        if kind == "plan":
            s.plan = ctx.plan_create(s.jobs)
    elif kind == "track":
        frames, s.feats = _track_inputs(case, seed)
        s.pyr = [fastgrid.Pyramid(case["width"], case["height"], case["levels"]) for _ in frames]
        for p, img in zip(s.pyr, frames):
            p.tensors[0][:, :case["width"]].copy_(img)
            ctx.pyr_build(p)
        s.q = torch.zeros((case["features"], 4), dtype=torch.float32, device="cuda")
        s.status = torch.zeros(case["features"], dtype=torch.int32, device="cuda")
    else:
        _prepare_frontend(s, case, seed)
    torch.cuda.synchronize()
    return s


def _prepare_frontend(s, case, seed):
    """Cameras whose first frame has been served: its pyramid is built and
    its features live; the second frame has arrived."""
    w, h, levels, cell, target = (case[k] for k in ("width", "height", "levels", "cell", "target"))
    count = case["cameras"]
    s.frames = [_Frames([(w, h, levels, cell)] * count) for _ in range(2)]
    s.feats = torch.zeros((count, target, 2), dtype=torch.float32, device="cuda")
    s.count = torch.full((count,), target, dtype=torch.int32, device="cuda")
    s.info = torch.zeros((count, 4), dtype=torch.int32, device="cuda")
    s.q = torch.zeros((count, target, 4), dtype=torch.float32, device="cuda")
    s.status = torch.zeros((count, target), dtype=torch.int32, device="cuda")
    for c in range(count):
        frames, feats = _camera_inputs(case, seed, c)
        for k in range(2):
            s.frames[k].fill(c, frames[k])
        s.feats[c].copy_(feats)
        s.ctx.pyr_build(s.frames[0].pyr[c])
    below = max(0, min(target, math.ceil(case["below"] * target)))
    P = fastgrid.ctypes.POINTER(fastgrid.fast_plane)
    s.detect, s.step = [], []
    for k in range(2):   # k: the frame that is current
        cur, prev = s.frames[k], s.frames[1 - k]
        s.detect.append(s.ctx.make_jobs((p, case["t"], case["n"], cell, g, fastgrid.FAST_SCORE_SADA)
                                        for p, g in zip(cur.pyr, cur.grid)))
        jobs = (fastgrid.fast_frontend_job * count)()
        for c in range(count):
            jobs[c] = fastgrid.fast_frontend_job(
                fastgrid.ctypes.cast(prev.pyr[c].planes, P), fastgrid.ctypes.cast(cur.pyr[c].planes, P), levels,
                cur.grid[c].ptr, cell, target, below, s.feats[c].data_ptr(), s.count[c:].data_ptr(),
                s.q[c].data_ptr(), s.status[c].data_ptr(), s.info[c].data_ptr())
        s.step.append(jobs)
    s.current = 1


# -------------------------------------------------------------------- pass

def _room(ctx, used):
    """Waits until few enough submissions are in flight, as the context has
    eight job tables and a submission uses `used` of them."""
    while sum(n for _, n in _in_flight) + used > 8:
        ctx.wait(_in_flight.popleft()[0])


def run(s):
    case, ctx = s.case, s.ctx
    if s.kind == "detect":
        ctx.detect(s.pyr, case["t"], case["n"], case["cell"], s.grid, score=s.score)
        return [s.grid.tensor] + s.pyr.tensors[1:]
    if s.kind == "plan":
        ctx.plan_launch(s.plan, ticket=False)
        return s.frames.outputs()
    if s.kind == "submit":
        _room(ctx, 2)
        _in_flight.append((ctx.submit(s.jobs), 2))
        return s.frames.outputs()
    if s.kind == "maps":
        ctx.score_maps(s.pyr, case["t"], case["n"], s.maps, score=s.score)
        ctx.nms_grid(s.maps, case["radius"], case["cell"], s.grid)
        return [s.grid.tensor] + s.maps.tensors + s.pyr.tensors[1:]
    if s.kind == "pyramid":
        ctx.pyr_build(s.pyr)
        return s.pyr.tensors[1:]
    if s.kind == "track":
        s.q.zero_()
        ctx.track(s.pyr[0], s.pyr[1], s.feats, s.q, s.status, mode=MODE, max_iter=MAX_ITER, eps=case["eps"])
        return [s.q, s.status]
    # the two frames take turns as the current one, so the features move
    # there and back
    _room(ctx, 2)
    cur = s.current
    ctx.submit(s.detect[cur])
    _in_flight.append((fastgrid.fast_frontend_step(ctx.handle, s.step[cur], len(s.step[cur]), MODE, MAX_ITER,
                                                   case["eps"]), 2))
    s.current = 1 - cur
    return [s.feats, s.count, s.info] + s.frames[cur].outputs()


# -------------------------------------------------------------------- work

def _upper_bytes(w, h, levels):
    return sum((w >> k) * (h >> k) for k in range(1, levels))


def _frame_bytes(w, h, levels, cell):
    return w * h + _upper_bytes(w, h, levels) + 8 * -(-w // cell) * -(-h // cell)


def _pixel_levels(w, h, levels):
    return w * h + _upper_bytes(w, h, levels)


def _track_work(w, h, levels, features):
    """Patches read once from both pyramids (at most the pyramids), and five
    Gauss-Newton steps a level of about 25 operations a patch pixel."""
    pixels = sum((16 if k < 2 else 8) ** 2 for k in range(levels))
    read = min(2 * _pixel_levels(w, h, levels),
               features * sum((18 if k < 2 else 10) ** 2 + (17 if k < 2 else 9) ** 2 for k in range(levels)))
    return {"bytes": read + features * (8 + 2 * 16 + 4), "flops": features * pixels * (70 + 5 * 25)}


def work(case):
    """Bytes read and written once; operations: for detection the four
    compass comparisons a pixel cannot do without, two sides each."""
    kind = case["kind"]
    if kind in ("plan", "submit"):
        mix = _mix(case)
        return {"bytes": sum(_frame_bytes(w, h, lv, c) for w, h, lv, _, _, c, _ in mix),
                "flops": sum(8 * _pixel_levels(w, h, lv) for w, h, lv, _, _, _, _ in mix)}
    w, h, levels = case["width"], case["height"], case["levels"]
    if kind == "pyramid":
        return {"bytes": _pixel_levels(w, h, levels), "flops": 4 * _upper_bytes(w, h, levels)}
    if kind == "track":
        return _track_work(w, h, levels, case["features"])
    frame = _frame_bytes(w, h, levels, case["cell"])
    if kind == "detect":
        return {"bytes": frame, "flops": 8 * _pixel_levels(w, h, levels)}
    if kind == "maps":
        # the maps are written by one entry point and read by the other
        r = 2 * case["radius"] + 1
        return {"bytes": frame + 4 * _pixel_levels(w, h, levels), "flops": (8 + 2 * r) * _pixel_levels(w, h, levels)}
    one = _track_work(w, h, levels, case["target"])
    return {"bytes": case["cameras"] * (frame + one["bytes"]),
            "flops": case["cameras"] * (8 * _pixel_levels(w, h, levels) + one["flops"])}


# ------------------------------------------------------------------- exact

def exact(case, seed):
    """The tracker's estimates in 64 bits; everything else is whole numbers."""
    if case["kind"] == "track":
        frames, feats = _track_inputs(case, seed)
        q, _ = _track64(frames[0], frames[1], case["levels"], feats.double(), case["eps"])
        return [q.cpu(), None]
    if case["kind"] == "frontend" and case["below"] <= 0.3:
        out = []
        for c in range(case["cameras"]):
            frames, feats = _camera_inputs(case, seed, c)
            q, status = _track64(frames[0], frames[1], case["levels"], feats.double(), case["eps"])
            kept = feats.double()[status == 0] + q[status == 0, :2]
            if len(kept) < math.ceil(case["below"] * case["target"]):
                return None   # a re-detection adds cell winners
            out.append(torch.cat([kept, feats.double()[len(kept):]]))   # entries past the live ones stay
        return [torch.stack(out).cpu(), None, None, None, None]
    return None


def _pyramid64(img, levels):
    out = [img.to(torch.int32)]
    for _ in range(1, levels):
        a = out[-1][:out[-1].shape[0] // 2 * 2, :out[-1].shape[1] // 2 * 2]
        out.append((a[0::2, 0::2] + a[0::2, 1::2] + a[1::2, 0::2] + a[1::2, 1::2] + 2) >> 2)
    return [v.double() for v in out]


def _sample(img, x, y):
    """Bilinear samples of img at positions inside it."""
    x0, y0 = x.floor().long().clamp(0, img.shape[1] - 2), y.floor().long().clamp(0, img.shape[0] - 2)
    ax, ay, flat = x - x0, y - y0, img.reshape(-1)
    i = y0 * img.shape[1] + x0
    top = (1 - ax) * flat[i] + ax * flat[i + 1]
    i = i + img.shape[1]
    return (1 - ay) * top + ay * ((1 - ax) * flat[i] + ax * flat[i + 1])


def _inside(p, img, lo, hi):
    """Where every sample from p + lo to p + hi has its four pixels."""
    h, w = img.shape
    return (p + lo >= 0).all(1) & (p[:, 0] + hi < w - 1) & (p[:, 1] + hi < h - 1)


def _patch(p, half):
    """The sample positions of the patch around each position."""
    o = torch.arange(2 * half, device=p.device, dtype=torch.float64) - half
    return p[:, :1] + o.repeat(2 * half), p[:, 1:] + o.repeat_interleave(2 * half)


def _steepest(img, p, half, gain):
    """The steepest-descent rows [gain dT/dx, gain dT/dy, T, 1] of each patch."""
    x, y = _patch(p, half)
    t = _sample(img, x, y)
    return torch.stack([gain * (_sample(img, x + 1, y) - _sample(img, x - 1, y)) / 2,
                        gain * (_sample(img, x, y + 1) - _sample(img, x, y - 1)) / 2, t, torch.ones_like(t)], 2)


def _cholesky(u):
    """The factor L of each feature's Hessian sum u u^T, and where a pivot
    falls to 1e-6 of its diagonal entry."""
    hess = torch.stack([(u * u[:, :, j:j + 1]).sum(1) for j in range(4)], 2)
    low, bad = torch.zeros_like(hess), torch.zeros(len(u), dtype=torch.bool, device=u.device)
    for i in range(4):
        for j in range(i + 1):
            v = hess[:, i, j] - (low[:, i, :j] * low[:, j, :j]).sum(1)
            if i == j:
                bad |= ~(v > 1e-6 * hess[:, i, i])
                low[:, i, i] = v.clamp(min=1e-300).sqrt()
            else:
                low[:, i, j] = v / low[:, j, j]
    return low, bad


def _solve(low, b):
    """d with L L^T d = b."""
    y, d = torch.zeros_like(b), torch.zeros_like(b)
    for i in range(4):
        y[:, i] = (b[:, i] - (low[:, i, :i] * y[:, :i]).sum(1)) / low[:, i, i]
    for i in reversed(range(4)):
        d[:, i] = (y[:, i] - (low[:, i + 1:, i] * d[:, i + 1:]).sum(1)) / low[:, i, i]
    return d


def _track64(tpl, img, levels, feats, eps):
    """Pyramidal Lucas-Kanade with translation, gain and offset (Section II-E)
    of all features at once, coarse to fine, from zero.  Status 0: tracked,
    1: the template patch leaves a level, 2: the warped patch does, 3: the
    Hessian is singular."""
    T, I = _pyramid64(tpl, levels), _pyramid64(img, levels)
    q = torch.zeros((len(feats), 4), dtype=torch.float64, device=feats.device)
    status = torch.zeros(len(feats), dtype=torch.int64, device=feats.device)
    for k in reversed(range(levels)):
        side, scale = 16 if k < 2 else 8, float(1 << k)
        half, p = side // 2, feats / scale
        live = status == 0
        status[live & ~_inside(p, T[k], -half - 1, half)] = 1
        live = status == 0
        if not live.any():
            break
        x, y = _patch(p[live], half)
        u = _steepest(T[k], p[live], half, 1.0 + q[live, 2:3])
        t = u[:, :, 2]
        factor, singular = _cholesky(u)
        at = live.nonzero()[:, 0]
        est = q[live].clone()
        est[:, :2] /= scale
        going = torch.ones(len(at), dtype=torch.bool, device=feats.device)
        for _ in range(MAX_ITER):
            lost = going & ~_inside(p[live] + est[:, :2], I[k], -half, half - 1)
            status[at[lost]] = 2
            going &= ~lost
            status[at[going & singular]] = 3
            going &= ~singular
            if not going.any():
                break
            a = going.nonzero()[:, 0]
            e = est[a]
            r = _sample(I[k], x[a] + e[:, :1], y[a] + e[:, 1:2]) - (1.0 + e[:, 2:3]) * t[a] - e[:, 3:]
            b = (u[a] * r[:, :, None]).sum(1)
            d = _solve(factor[a], b)
            est[a] = e + d * torch.tensor([-1.0, -1.0, 1.0, 1.0], dtype=torch.float64, device=feats.device)
            going[a[(d[:, :2] ** 2).sum(1) < eps * eps]] = False
        est[:, :2] *= scale
        q[at] = est
    return q, status
