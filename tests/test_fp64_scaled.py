"""FP64 counts from the iteration on twice the iterate: X' = (X^2 - Y^2)/2 + 2 Re C,
Y' = X Y + 2 Im C, test X^2 + Y^2 <= 16.

On the CPU, numpy's counts of that form equal the oracle's over constants with
zero, small and large parts and windows of every scale that it is given (no part
strictly between 0 and 2^-200).  On the GPU, images of those frames and of frames
it is not given equal the oracle's."""
import math
import random
from fractions import Fraction

import numpy as np
import pytest

import oracle

CS = [complex(-0.8, 0.156), complex(-1.0, 0.0), complex(0.0, 0.65), 0j, complex(-2.0, 0.0),
      complex(0.25, 2.0 ** -190), complex(2.0 ** -199, -0.7), complex(-0.75, 1e-17),
      complex(-1.7, 0.5), complex(1.2, 1.3)]
WINDOWS = [(-1.6, 1.6, -1.2, 1.2), (-1e-9, 3e-9, -2e-9, 2e-9), (0.1, 0.1 + 1e-15, -0.5, 0.5),
           (-1e200, 1.5e200, -1e190, 1e190), (-1e308, 5e307, -1e154, 2e154),
           (-1e-50, 1e-50, -1e-40, 3e-40), (-2.2, 0.9, -1.0, 1.0)]
UNDER = [(complex(0.1, 2.0 ** -1030), WINDOWS[0]), (complex(-0.5, 0.0), (-1e-300, 1e-300, -1, 1)),
         (complex(2.0 ** -400, 0.0), WINDOWS[0]), (0j, (-1e-160, 1e-160, -1e-160, 1e-160)),
         (complex(-1.0, 0.0), (-1.5, 1.5, -1e-310, 1e-310))]


def scaled_counts(c, win, w, h, cap, mandelbrot):
    jj, ii = np.meshgrid(np.arange(h), np.arange(w), indexing="ij")
    hx, hy = (win[1] - win[0]) / (2.0 * w), (win[3] - win[2]) / (2.0 * h)
    x = 0.5 * (win[0] + win[1]) + (2 * ii + 1 - w) * hx
    y = 0.5 * (win[2] + win[3]) - (2 * jj + 1 - h) * hy
    with np.errstate(all="ignore"):
        x, y = x + x, y + y
        cr, ci = np.full_like(x, c.real + c.real), np.full_like(x, c.imag + c.imag)
        if mandelbrot:
            cr, ci, x, y = x, y, np.zeros_like(x), np.zeros_like(y)
        out, inside = np.zeros(x.shape, np.int32), np.ones(x.shape, bool)
        for _ in range(cap):
            x2, y2 = x * x, y * y
            inside &= x2 + y2 <= 16.0
            out += inside
            # halving is exact here, so this is the fma
            x, y = (x2 - y2) * 0.5 + cr, x * y + ci
    return out


@pytest.mark.parametrize("win", WINDOWS)
def test_the_scaled_form_counts_alike(win):
    for c in CS:
        want = oracle.render(c, win, 41, 30, 150, "fp64")
        np.testing.assert_array_equal(scaled_counts(c, win, 41, 30, 150, False), want, err_msg=str(c))
    want = oracle.render(0j, win, 41, 29, 150, "fp64", "mandelbrot")
    np.testing.assert_array_equal(scaled_counts(0j, win, 41, 29, 150, True), want)


def test_a_shared_reciprocal_divides_correctly():
    """From a reciprocal good to an ulp, one more step and one correction give
    the rounded quotient, but for a divisor with every bit set (exact fma through
    fractions)."""
    def fma(a, b, c):
        v = Fraction(a) * Fraction(b) + Fraction(c)
        return v.numerator / v.denominator
    rng = random.Random(1)
    for k in range(6000):
        m = rng.getrandbits(52)
        if k % 8 == 0:
            m = rng.choice([0, 1, 2, (1 << 52) - 2, (1 << 52) - 3, 1 << 51, (1 << 51) - 1])
        q = math.ldexp((1 << 52) | m, rng.randint(-500, 16) - 52)
        a = rng.uniform(-1, 1) * 2.0 ** rng.randint(-400, 8)
        if m == (1 << 52) - 1:
            continue
        for off in (-1, 0, 1):
            r = 1.0 / q
            r += off * math.ulp(r)
            r = fma(fma(-q, r, 1.0), r, r)
            t = a * r
            assert fma(fma(-q, t, a), r, t) == a / q


@pytest.mark.gpu
@pytest.mark.parametrize("degree", [2, 3, 4, 8])
def test_rational_quotients_equal_the_oracle(degree):
    """Both quotients of the rational map come from one reciprocal: windows on the
    pole (0, and the next to it), divisors from 2^16 down past 2^-500, divisors
    that are powers of two and the like (exact orbits), real and imaginary
    constants, and parts too small for the shared form, in every schedule of blocks."""
    import torch
    import paper_1611_03079_amd as jr
    from workloads import Frame
    rng = np.random.default_rng(degree)
    wins = [(-1.6, 1.6, -1.2, 1.2), (-1.0, 1.0, -1.0, 1.0), (-1e-3, 1e-3, -1e-3, 1.1e-3),
            (-1e-40, 1e-40, -1e-40, 2e-40), (-1e-90, 1e-90, -2e-90, 1e-90),
            (-1e-300, 1e-300, -1, 1), (0.5, 0.5 + 2.0 ** -30, 0.25, 0.75)]
    cases = [(0j, 0.25 + 0j), (-0.5 + 0j, -0.125 + 0j), (0.3j, 0.01j), (0.25 + 0.25j, 1e-30 + 0j),
             (-0.1 + 0.1j, complex(2.0 ** -300, 0.0)), (complex(2.0 ** -260, 0.4), -0.01 + 0j)]
    cases += [(complex(*rng.uniform(-0.7, 0.7, 2)), complex(*rng.uniform(-0.05, 0.05, 2)))
              for _ in range(10)]
    frames = [Frame(c, w, 37, 26, 70, "fp64", "julia", degree, lam) for c, lam in cases
              for w in wins]
    want = [oracle.render(f.c, f.window, 37, 26, 70, "fp64", "julia", degree, f.lam)
            for f in frames]
    for sched in (None, jr.Schedule(64, 8, 4, 0, 8, 0, 16, "cost", "rows", 8),
                  jr.Schedule(20, 6, 8, 0, 16, 1, 16, "table", "rows", 4)):
        _, views = jr.render_batch(frames, sched)
        torch.cuda.synchronize()
        for f, v, w in zip(frames, views, want):
            np.testing.assert_array_equal(v.cpu().numpy(), w, err_msg=str(f))


@pytest.mark.gpu
def test_images_at_every_scale_equal_the_oracle():
    import torch
    import paper_1611_03079_amd as jr
    from workloads import Frame
    frames = [Frame(c, win, 41, 30, 150, "fp64") for c in CS for win in WINDOWS]
    frames += [Frame(0j, win, 41, 29, 300, "fp64", "mandelbrot") for win in WINDOWS]
    frames += [Frame(c, win, 41, 30, 150, "fp64") for c, win in UNDER]
    frames += [Frame(0j, win, 41, 30, 150, "fp64", "mandelbrot") for _, win in UNDER]
    want = [oracle.render(f.c, f.window, f.width, f.height, f.max_iter, "fp64", f.mode)
            for f in frames]
    for sched in (None, jr.Schedule(64, 16, 8, 0, 16, 0, 16, "cost", "rows", 8, 32),
                  jr.Schedule(64, 8, 4, 1, 16, 1, 16, "table", "rows", 16, 0)):
        _, views = jr.render_batch(frames, sched)
        torch.cuda.synchronize()
        for f, v, w in zip(frames, views, want):
            np.testing.assert_array_equal(v.cpu().numpy(), w, err_msg=str(f))
    for f, w in zip(frames, want):
        got = jr.render(f.c, f.window, f.width, f.height, f.max_iter, "fp64", mode=f.mode)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(got.cpu().numpy(), w, err_msg=str(f))
