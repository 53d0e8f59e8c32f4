"""Workloads by which the renderer's speed is measured, as a user's program runs them.

Each case is one call (or one replay of a prepared plan) through the public
entry points of ``paper_1611_03079_amd``.  Four kinds cover the uses of an
escape-time renderer:

  image   one image through ``render``: thumbnails, the paper's 512^2 image,
          a screen-sized coloured view, 4096^2 stills;
  path    an animation: frames along a path of constants, prepared once as a
          ``Plan`` with the shipped autotuned schedule and replayed from its graph;
  zoom    an animation into the Mandelbrot set, the window shrinking per frame;
  batch   frames of unlike sizes, caps and arithmetics in one ``render_batch``
          call with the library's default schedule: an uneven job, or the
          requests of interactive users as a server finds them waiting.

A seed moves every constant a little (and a batch's windows with it), so
another seed is another picture of about the same cost.
"""
import math
import random

import numpy as np
import torch

import paper_1611_03079_amd as jr
import workloads as wl
from paper_1611_03079_amd import autotune
from paper_1611_03079_amd.serve import PrecisionPolicy

FULL_HD = (-1.78, 1.78, -1.0, 1.0)


def listed():
    return [
        # a thumbnail: the call itself is what costs
        dict(name="thumbnail_100_fp64", kind="image", width=100, height=100, cap=100,
             dtype="fp64", c_re=-0.8, c_im=0.156, x=0.0, y=0.0, extent=3.0, colours=0),
        # the paper's kind of image: a few hundred pixels a side, FP64, cap 100
        dict(name="image_512_fp64", kind="image", width=512, height=512, cap=100,
             dtype="fp64", c_re=-0.8, c_im=0.156, x=0.0, y=0.0, extent=3.0, colours=0),
        # an exploring user's screen: part of the set, coloured by the kernel
        dict(name="screen_1080_fp32_coloured", kind="image", width=1920, height=1080, cap=500,
             dtype="fp32", c_re=-0.7269, c_im=0.1889, x=0.31, y=0.17, extent=0.8, colours=256),
        # a large still, short arithmetic, high cap
        dict(name="still_4096_fp32", kind="image", width=4096, height=4096, cap=1000,
             dtype="fp32", c_re=-0.66258, c_im=-0.42746, x=0.0, y=0.0, extent=3.2, colours=0),
        # a large still in the defining arithmetic, the paper's cap
        dict(name="still_4096_fp64", kind="image", width=4096, height=4096, cap=100,
             dtype="fp64", c_re=-0.72054, c_im=-0.32024, x=0.0, y=0.0, extent=3.2, colours=0),
        # the headline animation: one turn of the constant around the circle |C| = 0.7885
        dict(name="path_256_fp32", kind="path", frames=256, width=1920, height=1080, cap=100,
             dtype="fp32", degree=2, lam=0.0),
        # the same in the defining arithmetic, a shorter clip
        dict(name="path_64_fp64", kind="path", frames=64, width=1920, height=1080, cap=100,
             dtype="fp64", degree=2, lam=0.0),
        # the further functions: Z^3 + C, and the rational map Z^2 + C + lambda / Z^2
        dict(name="path_cubic_32_fp32", kind="path", frames=32, width=1920, height=1080, cap=100,
             dtype="fp32", degree=3, lam=0.0),
        dict(name="path_rational_32_fp64", kind="path", frames=32, width=1920, height=1080,
             cap=100, dtype="fp64", degree=2, lam=0.002),
        # a zoom into the seahorse valley, cap 1000
        dict(name="zoom_24_fp64", kind="zoom", frames=24, width=1920, height=1080, cap=1000,
             dtype="fp64", w0=3.0, w1=1e-5),
        # an uneven job: sides 256..4096, caps 100/500/2000, FP32 and float-float
        dict(name="uneven_96_fp32_ff", kind="batch", recipe="uneven", stream=0, frames=96),
        # what a server finds waiting: windows from 1e-9 to 3 wide, caps 100..5000,
        # screen sizes, the arithmetic by the serving policy
        dict(name="requests_24", kind="batch", recipe="requests", stream=7, frames=24),
    ]


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    kind = rng.choice(("image", "image", "path", "zoom", "batch"))
    if kind == "image":
        w = int(round(_log_uniform(rng, 10, 6000)))
        h = max(1, min(6000, int(round(w * _log_uniform(rng, 0.4, 1.6)))))
        c = wl.sample_c_disk(wl.SplitMix64(rng.getrandbits(60)))
        if rng.random() < 0.4:
            t = rng.uniform(0.0, 2.0 * math.pi)
            c = complex(0.7885 * math.cos(t), 0.7885 * math.sin(t))
        part = rng.random() < 0.4
        dtype = rng.choice(("fp32", "fp64", "ff") if not part else ("fp32", "fp64"))
        return dict(kind="image", width=w, height=h, cap=rng.choice((100, 100, 250, 1000)),
                    dtype=dtype, c_re=c.real, c_im=c.imag,
                    x=rng.uniform(-0.6, 0.6) if part else 0.0,
                    y=rng.uniform(-0.5, 0.5) if part else 0.0,
                    extent=_log_uniform(rng, 0.02, 1.5) if part else rng.uniform(2.6, 3.6),
                    colours=rng.choice((0, 0, 101, 256)))
    if kind == "path":
        what = rng.choice(("quadratic", "quadratic", "cubic", "rational"))
        dtype = {"cubic": "fp32", "rational": rng.choice(("fp32", "fp64"))}.get(
            what, rng.choice(("fp32", "fp64", "ff")))
        most = {"fp32": 128, "fp64": 64, "ff": 16}[dtype] if what == "quadratic" else 32
        return dict(kind="path", frames=rng.randint(4, most), width=rng.randint(320, 1920),
                    height=rng.randint(200, 1080), cap=rng.choice((100, 100, 128)), dtype=dtype,
                    degree=3 if what == "cubic" else 2, lam=0.002 if what == "rational" else 0.0)
    if kind == "zoom":
        return dict(kind="zoom", frames=rng.randint(4, 24), width=rng.randint(320, 1920),
                    height=rng.randint(200, 1080), cap=rng.choice((500, 1000)), dtype="fp64",
                    w0=3.0, w1=_log_uniform(rng, 1e-6, 1e-3))
    recipe = rng.choice(("uneven", "requests"))
    return dict(kind="batch", recipe=recipe, stream=rng.randint(1, 10 ** 6),
                frames=rng.randint(8, 64) if recipe == "uneven" else rng.randint(4, 24))


def _frames(case, seed):
    """The frames of a case, from the recipes that the benchmarks and tests use."""
    rng = random.Random(seed)
    kind = case["kind"]
    if kind == "image":
        c = complex(case["c_re"] + rng.uniform(-5e-4, 5e-4), case["c_im"] + rng.uniform(-5e-4, 5e-4))
        hw = 0.5 * case["extent"]
        hh = hw * case["height"] / case["width"]
        win = (case["x"] - hw, case["x"] + hw, case["y"] - hh, case["y"] + hh)
        return [wl.Frame(c, win, case["width"], case["height"], case["cap"], case["dtype"])]
    if kind == "path":
        n, turn = case["frames"], rng.uniform(0.0, 2.0 * math.pi / case["frames"])
        cubic = case["degree"] == 3
        out = []
        for k in range(n):
            t = 2.0 * math.pi * k / n + turn
            r = 0.6 if cubic else 0.7885
            win = (-1.6, 1.6, -0.9, 0.9) if cubic else FULL_HD
            lam = None
            if case["lam"]:
                lam = complex(case["lam"] * math.cos(t), -case["lam"] * math.sin(t))
            out.append(wl.Frame(complex(r * math.cos(t), r * math.sin(t)), win, case["width"],
                                case["height"], case["cap"], case["dtype"], "julia",
                                case["degree"], lam))
        return out
    if kind == "zoom":
        s = 1.0 + rng.uniform(-0.02, 0.02)
        return wl.mandelbrot_zoom(case["frames"], case["w0"] * s, case["w1"] * s, case["width"],
                                  case["height"], case["cap"], case["dtype"])
    if case["recipe"] == "uneven":
        frames = wl.uneven_batch(case["stream"], case["frames"])
        for f in frames:
            f.c += complex(rng.uniform(-5e-4, 5e-4), rng.uniform(-5e-4, 5e-4))
        return frames
    frames = [r.frame for r in wl.serving_stream(case["stream"], 200.0, case["frames"])]
    policy = PrecisionPolicy()
    for f in frames:
        w, h = f.window[1] - f.window[0], f.window[3] - f.window[2]
        f.dtype = policy.pick(w, f.max_iter)
        f.c += complex(rng.uniform(-5e-4, 5e-4), rng.uniform(-5e-4, 5e-4))
        dx, dy = rng.uniform(-0.02, 0.02) * w, rng.uniform(-0.02, 0.02) * h
        f.window = (f.window[0] + dx, f.window[1] + dx, f.window[2] + dy, f.window[3] + dy)
    return frames


def _palette(case):
    k = np.arange(case["colours"], dtype=np.uint64)
    return (k * np.uint64(2654435761) % np.uint64(1 << 31)).astype(np.int32)


def _tuned(case):
    """The shipped schedule of the animation this case is one of."""
    if case["kind"] == "zoom":
        name = "mandelbrot_zoom_fp64"
    elif case["degree"] == 3:
        name = "general_deg3_fp32"
    elif case["lam"]:
        name = "rational_deg2_" + case["dtype"]
    else:
        name = "parameter_path_" + case["dtype"]
    return jr.Schedule(**autotune.load_cache()["_workloads"][name]["schedule"])


def prepare(case, seed):
    frames = _frames(case, seed)
    state = {"kind": case["kind"], "frames": frames}
    if case["kind"] == "image":
        f = frames[0]
        state["out"] = torch.empty((f.height, f.width), dtype=torch.int32, device="cuda")
        state["palette"] = torch.from_numpy(_palette(case)).cuda() if case["colours"] else None
    elif case["kind"] in ("path", "zoom"):
        state["plan"] = jr.Plan(frames, _tuned(case))
        state["plan"].capture()
    else:
        state["arena"] = torch.empty(sum(f.pixels for f in frames), dtype=torch.int32,
                                     device="cuda")
    return state


def run(state):
    if state["kind"] == "image":
        f = state["frames"][0]
        return jr.render(f.c, f.window, f.width, f.height, f.max_iter, f.dtype,
                         out=state["out"], palette=state["palette"])
    if state["kind"] in ("path", "zoom"):
        state["plan"].replay()
        return state["plan"].arena
    arena, _ = jr.render_batch(state["frames"], arena=state["arena"])
    return arena


# Operations of one iteration with its test: the quadratic map's eight; a
# double-word iteration; two more complex products' worth for the cubic map; the
# rational map's product, norm, quotient and sums.
def _flops_per_iteration(f):
    if f.lam is not None:
        return 26.0
    return {2: 8.0, 3: 17.0}[f.degree] * (9.0 if f.dtype == "ff" else 1.0)


def _iterate(x, y, cr, ci, f):
    if f.degree == 2 and f.lam is None:
        return (x * x - y * y) + cr, ((x + x) * y) + ci
    wr, wi = x, y
    for _ in range(f.degree - 1):
        wr, wi = wr * x - wi * y, wr * y + wi * x
    if f.lam is None:
        return wr + cr, wi + ci
    lr, li = f.lam.real, f.lam.imag
    q = wr * wr + wi * wi
    return (wr + cr) + (lr * wr + li * wi) / q, (wi + ci) + (li * wr - lr * wi) / q


def _starts(f, ii, jj):
    """Pixel centres of columns ii and rows jj, in 64 bits."""
    w = f.window
    x = 0.5 * (w[0] + w[1]) + (2 * ii + 1 - f.width) * ((w[1] - w[0]) / (2.0 * f.width))
    y = 0.5 * (w[2] + w[3]) - (2 * jj + 1 - f.height) * ((w[3] - w[2]) / (2.0 * f.height))
    return x, y


def work(case):
    """Bytes: one 32-bit store per pixel.  Operations: the iterations that the
    escaping pixels take before they leave the disc, from a grid of samples.  A
    pixel that stays is counted as free, since how many steps show that it stays
    depends on the method, and an even map on a window about 0 is counted once for
    each pair of opposite pixels, whose orbits are each other's negatives."""
    frames = _frames(case, 0)
    pixels = sum(f.pixels for f in frames)
    flops = 0.0
    some = frames[:: max(1, len(frames) // 24)]
    for f in some:
        ii, jj = np.meshgrid((np.arange(48) + 0.5) * f.width / 48 - 0.5,
                             (np.arange(27) + 0.5) * f.height / 27 - 0.5)
        x, y = _starts(f, ii.ravel(), jj.ravel())
        cr, ci = f.c.real, f.c.imag
        if f.mode == "mandelbrot":
            cr, ci, x, y = x, y, np.zeros_like(x), np.zeros_like(y)
        n, inside, steps = x.size, np.ones(x.size, bool), 0.0
        with np.errstate(all="ignore"):
            for k in range(min(f.max_iter, 300)):
                left = inside & ~(x * x + y * y <= 4.0)
                steps += k * int(left.sum())
                inside &= ~left
                x, y = _iterate(x, y, cr, ci, f)
        w = f.window
        about0 = w[0] == -w[1] and w[2] == -w[3] and f.mode == "julia" and f.degree % 2 == 0
        flops += f.pixels * (steps / n) * _flops_per_iteration(f) * (0.5 if about0 else 1.0)
    flops *= pixels / sum(f.pixels for f in some)
    return {"bytes": 4.0 * pixels, "flops": flops}


def _counts(f):
    """Counts of a frame in 64 bits, each operation rounded, with plain torch."""
    jj, ii = torch.meshgrid(torch.arange(f.height, device="cuda", dtype=torch.float64),
                            torch.arange(f.width, device="cuda", dtype=torch.float64),
                            indexing="ij")
    x, y = _starts(f, ii.reshape(-1), jj.reshape(-1))
    cr, ci = torch.full_like(x, f.c.real), torch.full_like(x, f.c.imag)
    if f.mode == "mandelbrot":
        cr, ci, x, y = x, y, torch.zeros_like(x), torch.zeros_like(y)
    out = torch.full((x.numel(),), f.max_iter, dtype=torch.int32, device="cuda")
    at = torch.arange(x.numel(), device="cuda")
    for k in range(f.max_iter):
        inside = x * x + y * y <= 4.0
        if k % 8 == 0 or k < 8:  # only now and then: finding the survivors waits for the GPU
            out[at[~inside]] = torch.minimum(out[at[~inside]], torch.tensor(k, device="cuda", dtype=torch.int32))
            at, x, y, cr, ci = at[inside], x[inside], y[inside], cr[inside], ci[inside]
            if at.numel() == 0:
                break
        else:
            out[at] = torch.where(inside, out[at], torch.minimum(out[at], torch.full_like(out[at], k)))
        x, y = _iterate(x, y, cr, ci, f)
    return out


def exact(case, seed):
    """The counts in 64 bits; where the case renders in a shorter arithmetic, the
    counts that it approximates."""
    frames = _frames(case, seed)
    if sum(f.pixels * (40 + 0.3 * f.max_iter) for f in frames) > 3e10:
        return None
    counts = torch.cat([_counts(f) for f in frames])
    if case["kind"] != "image":
        return counts
    f = frames[0]
    if case["colours"]:
        pal = torch.from_numpy(_palette(case)).cuda()
        counts = pal[torch.clamp(counts, max=case["colours"] - 1).long()]
    return counts.view(f.height, f.width)
