"""FP64 frames with a part of their constants or window between 0 and 2^-200, which
keep the plain form of the iteration and of the quotient: they run in blocks, with
traps and repeats, like others, and equal the oracle alone and among others."""
import time

import numpy as np
import pytest

import oracle
from workloads import Frame

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_1611_03079_amd as jr  # noqa: E402

W = (-1.6, 1.6, -1.2, 1.2)
TINY = [Frame(complex(-0.7269, 1e-70), W, 131, 90, 300, "fp64"),
        Frame(complex(2.0 ** -400, 0.0), W, 131, 90, 150, "fp64"),
        Frame(complex(-0.1, 1e-300), (-1.6, 1.5, -1.2, 1.2), 70, 61, 400, "fp64"),
        Frame(complex(1.7, 1e-100), W, 64, 33, 100, "fp64"),
        Frame(complex(1.95, 1e-100), W, 64, 33, 100, "fp64"),
        Frame(complex(-0.5, 0.0), (-1e-300, 1e-300, -1, 1), 41, 30, 200, "fp64"),
        Frame(0j, (-1e-65, 1e-65, 0.8, 1.0), 90, 61, 500, "fp64", "mandelbrot"),
        Frame(0j, (-2.0, 1.0, -1e-90, 1e-90), 90, 61, 500, "fp64", "mandelbrot"),
        Frame(complex(0.0, 1e-70), W, 60, 47, 90, "fp64", "julia", 2, 0.002 + 0j),
        Frame(0.1 + 0.1j, W, 60, 47, 90, "fp64", "julia", 3, complex(0.002, 1e-80))]
OTHERS = [Frame(-0.8 + 0.156j, W, 80, 50, 100, dt) for dt in ("fp64", "fp32", "ff")] + \
         [Frame(0.3 + 0.2j, W, 80, 50, 100, "fp64", "julia", 3),
          Frame(0j, (-2.3, 0.9, -1.2, 1.25), 80, 50, 300, "fp64", "mandelbrot")]


def image(f):
    return oracle.render(f.c, f.window, f.width, f.height, f.max_iter, f.dtype, f.mode, f.degree,
                         f.lam)


@pytest.mark.parametrize("persistent", [0, 1])
def test_tiny_parts_equal_the_oracle(persistent):
    pal = np.arange(77, dtype=np.uint32) * np.uint32(2654435)
    for frames in [[f] for f in TINY] + [TINY, TINY[:8], OTHERS + TINY[:8], OTHERS + TINY]:
        want = [image(f) for f in frames]
        for unroll, defer in ((8, 0), (4, 1)):
            sched = jr.Schedule(64, 8, unroll, defer, 16, persistent, 16, "cost", "rows", 8, 24)
            plan = jr.Plan(frames, sched)
            done = torch.zeros(len(frames), dtype=torch.int32, device="cuda")
            for counted in (None, done):
                plan.arena.fill_(-1)
                plan.set_progress(counted)
                plan.launch()
                torch.cuda.synchronize()
                for f, v, w in zip(frames, plan.views, want):
                    np.testing.assert_array_equal(v.cpu().numpy(), w, err_msg=str(f))
            assert done.cpu().tolist() == [f.pixels for f in frames]
            plan.close()
            _, views = jr.render_batch(frames, sched, palette=torch.from_numpy(
                pal.view(np.int32).copy()).cuda())
            torch.cuda.synchronize()
            for f, v, w in zip(frames, views, want):
                np.testing.assert_array_equal(v.cpu().numpy().view(np.uint32),
                                              oracle.colorize(w, pal), err_msg=str(f))


def test_a_path_with_a_tiny_window_equals_the_oracle():
    p = jr.CardioidPath(complex(np.cos(0.5), np.sin(0.5)), 4.5, 0.05, (-1e-70, 1.5e-70, -1.2, 1.2),
                        4, 60, 50, 150, "fp64")
    _, views = jr.render_cardioid_path(p, jr.Schedule(64, 8, 8, 0, 16, 0, 16, "cost", "rows", 8))
    torch.cuda.synchronize()
    for k, v in enumerate(views):
        c = oracle.cardioid_constant(p.step, p.a0, p.da, k)
        np.testing.assert_array_equal(v.cpu().numpy(), oracle.render(
            c, p.window, 60, 50, 150, "fp64"), err_msg=str(k))


def test_a_tiny_part_does_not_cost_the_blocks():
    """Eight frames of 1024x768, cap 500, most of each in a trap: Im C = 1e-70 against
    Im C = 0.  41 and 32 us; tested on every iteration up to the cap, 985."""
    def best(im):
        plan = jr.Plan([Frame(complex(-0.7269 + 0.001 * k, im), W, 1024, 768, 500, "fp64")
                        for k in range(8)],
                       jr.Schedule(64, 16, 8, 0, 16, 0, 16, "cost", "rows", 8, 32))
        times = []
        for _ in range(10):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            for _ in range(5):
                plan.launch()
            torch.cuda.synchronize()
            times.append(time.perf_counter() - t0)
        plan.close()
        return min(times)
    assert best(1e-70) < 4 * best(0.0)
