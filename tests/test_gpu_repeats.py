"""Orbits that the rows kernel ends because an iterate came back to a point it
had been at, and the tiles of Mandelbrot views that reach beyond |C| = 1.9,
against the oracle: caps about the least that is looked at and longer ones,
every arithmetic, the Mandelbrot set's first bulbs, constants without a usable
trap (parabolic, or of too long a period), rational and general maps."""
import numpy as np
import pytest

import oracle
from workloads import Frame

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_1611_03079_amd as jr  # noqa: E402

WHOLE = (-2.3, 0.9, -1.2, 1.25)
FRAMES = [(WHOLE, 0j, "mandelbrot", 2, None, 600),
          ((-1.95, -1.7, -0.1, 0.12), 0j, "mandelbrot", 2, None, 257),
          ((-1.42, -1.2, -0.1, 0.1), 0j, "mandelbrot", 2, None, 900),
          ((-0.3, 0.0, 0.6, 0.85), 0j, "mandelbrot", 2, None, 129),
          ((0.2, 0.4, 0.4, 0.6), 0j, "mandelbrot", 2, None, 400),
          (WHOLE, 0j, "mandelbrot", 3, None, 300),
          ((-1.6, 1.6, -1.2, 1.2), 0.25 + 0j, "julia", 2, None, 700),
          ((-1.6, 1.6, -1.2, 1.2), -0.75 + 0j, "julia", 2, None, 500),
          ((-1.5, 1.6, -1.2, 1.2), -0.1011 + 0.9563j, "julia", 2, None, 500),
          ((-1.6, 1.5, -1.2, 1.2), -0.5125 + 0.5213j, "julia", 2, None, 400),
          ((-1.4, 1.4, -1.2, 1.2), 0.1 + 0.1j, "julia", 2, -0.001 + 0.001j, 400),
          ((-1.4, 1.4, -1.2, 1.2), -0.2 + 0.05j, "julia", 3, 0.002 + 0j, 300)]


@pytest.mark.parametrize("dtype", ["fp32", "fp64", "ff"])
def test_repeated_iterates_count_the_cap(dtype):
    frames = [Frame(c, win, 150, 101, cap, dtype, mode, deg, lam)
              for win, c, mode, deg, lam, cap in FRAMES if not (lam and dtype == "ff")]
    want = [oracle.render(f.c, f.window, f.width, f.height, f.max_iter, f.dtype, f.mode, f.degree,
                          f.lam) for f in frames]
    assert all((w == f.max_iter).sum() > 100 for w, f in zip(want[:6], frames[:6]))
    kinds = {"all": lambda f: True, "quadratic": lambda f: f.degree == 2 and f.lam is None,
             "polynomial": lambda f: f.lam is None}
    for sched in (jr.Schedule(64, 8, 8, 0, 8, 0, 16, "table", "rows", 8, 64),
                  jr.Schedule(64, 64, 4, 0, 32, 0, 16, "cost", "rows", 4, 0),
                  jr.Schedule(33, 5, 8, 1, 16, 1, 16, "cost", "rows", 16, 16), None):
        for name, pick in kinds.items():
            some = [k for k, f in enumerate(frames) if pick(f)]
            _, views = jr.render_batch([frames[k] for k in some], sched)
            torch.cuda.synchronize()
            for k, v in zip(some, views):
                np.testing.assert_array_equal(v.cpu().numpy(), want[k],
                                              err_msg="%s %s" % (name, frames[k]))
