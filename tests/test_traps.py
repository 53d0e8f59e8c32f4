"""Traps: discs about an attracting cycle that no orbit leaves, in which the rows
kernel ends an orbit with the cap as its count.

On the CPU: orbits started anywhere in the discs that the kernel tests run to
the cap in the oracle, in every arithmetic and degree.  On the GPU: images of
constants with cycles of several periods, of constants near the border of such
regions and of constants without a cycle equal the oracle's."""
import cmath
import ctypes
import math
import os
import subprocess

import numpy as np
import pytest

import oracle
from workloads import Frame

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_1611_03079_amd", "csrc")


@pytest.fixture(scope="module")
def find_trap(tmp_path_factory):
    d = tmp_path_factory.mktemp("trap")
    src = d / "t.cpp"
    src.write_text('#include "julia_trap.h"\n'
                   'extern "C" int find(double a, double b, int d, float* o, int* s) {\n'
                   '    return jr::find_trap(a, b, d, o, o + 1, o + 2, o + 3, s); }\n')
    lib = str(d / "t.so")
    subprocess.run(["g++", "-O2", "-ffp-contract=off", "-shared", "-fPIC", "-I", CSRC, str(src),
                    "-o", lib], check=True)
    fn = ctypes.CDLL(lib).find

    def call(c, degree=2):
        out, steps = (ctypes.c_float * 4)(), ctypes.c_int()
        p = fn(ctypes.c_double(c.real), ctypes.c_double(c.imag), degree, out, ctypes.byref(steps))
        return p, tuple(out), steps.value
    return call


def kernel_discs(p, disc, c, degree):
    """The discs as the kernel forms them, in binary32."""
    f = np.float32
    x, y, r, r1 = (f(v) for v in disc)
    out = []
    for _ in range(p):
        out.append((x, y, r * f(0.99) - f(1e-5)))
        m = np.sqrt(x * x + y * y)
        wr, wi, p0, p1 = x, y, m, m + r
        for _ in range(1, degree):
            wr, wi = wr * x - wi * y, wr * y + wi * x
            p0, p1 = p0 * m, p1 * (m + r)
        x, y, r = wr + f(c.real), wi + f(c.imag), r1 if p == 2 else p1 - p0
    return out


@pytest.mark.parametrize("degree", [2, 3, 4, 5, 8])
def test_orbits_started_in_the_discs_never_escape(find_trap, degree):
    rng = np.random.default_rng(degree)
    periods, tried = set(), 0
    while tried < (150 if degree == 2 else 50):
        c = complex(rng.uniform(-1.6, 0.6), rng.uniform(-1.1, 1.1))
        if abs(c) > 1.9:
            continue
        p, disc, _ = find_trap(c, degree)
        if p == 0 or (p == 1 and rng.random() < 0.8):
            continue
        tried += 1
        periods.add(p)
        for x, y, r in kernel_discs(p, disc, c, degree):
            assert r > 0
            for a in rng.uniform(0, 2 * math.pi, 3):
                z = complex(float(x) + 0.9999 * float(r) * math.cos(a),
                            float(y) + 0.9999 * float(r) * math.sin(a))
                for dt in ("fp32", "fp64", "ff"):
                    n = 300 if dt == "ff" else 1500
                    d = None if degree == 2 else degree
                    assert oracle.count(z, c, n, dt, degree=d) == n, (c, degree, p, z, dt)
    assert len(periods) >= 3


def test_no_trap_without_an_attracting_cycle(find_trap):
    """Constants outside the Mandelbrot set, and the steps of their critical
    orbits (the oracle's Mandelbrot counts, Z_0 = 0)."""
    rng = np.random.default_rng(1)
    for _ in range(300):
        c = complex(rng.uniform(-2, 1), rng.uniform(-1.3, 1.3))
        p, _, steps = find_trap(c)
        n = oracle.count(0j, c, 512)
        if n < 512:
            assert p == 0 and steps == n
        elif p == 0:
            assert steps == 512
    for c in (0.25 + 0j, -2 + 0j, 1j):  # parabolic, and bounded without attraction
        assert find_trap(c)[0] == 0



CONSTANTS = [(2, 0.1 + 0.1j), (2, 0.2495 + 0j), (2, -0.7495 + 0j), (2, -1 + 0.1j),
             (2, -0.1225 + 0.7449j), (2, 0.282 + 0.53j), (2, -0.504 + 0.563j),
             (2, -1.3107 + 0j), (2, -1.7549 + 0j), (2, 0.3 + 0.6j), (2, -0.8 + 0.156j),
             (3, 0.2 + 0.1j), (3, 0.1 + 0.9j), (4, -0.4 + 0.2j), (5, 0.2 - 0.3j), (8, 0.3 + 0.1j)]


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["fp32", "fp64", "ff"])
def test_images_with_traps_equal_the_oracle(dtype):
    """Whole sets, windows off 0, windows inside one disc, caps at the shortest
    that are trapped and longer ones, every drain of the rows kernel."""
    import torch
    import paper_1611_03079_amd as jr
    frames = []
    for k, (deg, c) in enumerate(CONSTANTS):
        for win, cap in (((-1.6, 1.6, -1.2, 1.2), (100, 33, 300)[k % 3]),
                         ((-0.3, 0.5, -0.41, 0.2), (32, 150, 31)[k % 3])):
            frames.append(Frame(c, win, 160, 107, cap, dtype, "julia", deg))
    want = [oracle.render(f.c, f.window, f.width, f.height, f.max_iter, f.dtype, f.mode, f.degree)
            for f in frames]
    quad = [k for k, f in enumerate(frames) if f.degree == 2]
    for sched in (None, jr.Schedule(64, 16, 8, 0, 16, 0, 16, "cost", "rows", 1),
                  jr.Schedule(64, 64, 4, 0, 16, 0, 16, "table", "rows", 32, 128),
                  jr.Schedule(37, 6, 4, 1, 64, 1, 16, "cost", "rows", 8, 0),
                  jr.Schedule(64, 32, 8, 1, 8, 0, 16, "cost", "rows", 4, 16)):
        for some in (range(len(frames)), quad):
            _, views = jr.render_batch([frames[k] for k in some], sched)
            torch.cuda.synchronize()
            for k, v in zip(some, views):
                np.testing.assert_array_equal(v.cpu().numpy(), want[k], err_msg=str(frames[k]))
    f = frames[0]
    got = jr.render(f.c, f.window, f.width, f.height, f.max_iter, f.dtype)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(got.cpu().numpy(), want[0])


@pytest.mark.gpu
def test_a_cardioid_path_with_traps_equals_the_oracle():
    """The device looks for the traps of a generated path's frames itself."""
    import torch
    import paper_1611_03079_amd as jr
    step = cmath.exp(2j * math.pi / 24)
    path = jr.CardioidPath(step, 4.6, 0.05, (-1.6, 1.6, -1.2, 1.2), 24, 160, 107, 150, "fp32")
    plan = jr.Plan.cardioid(path, jr.Schedule(64, 16, 8, 0, 16, 0, 16, "cost", "rows", 8, 32))
    plan.launch()
    torch.cuda.synchronize()
    for k, v in enumerate(plan.views):
        c = oracle.cardioid_constant(step, 4.6, 0.05, k)
        want = oracle.render(c, path.window, 160, 107, 150, "fp32")
        np.testing.assert_array_equal(v.cpu().numpy(), want, err_msg="frame %d" % k)
    plan.close()


@pytest.fixture(scope="module")
def settles(tmp_path_factory):
    d = tmp_path_factory.mktemp("settles")
    src = d / "s.cpp"
    src.write_text('#include "julia_trap.h"\n'
                   'extern "C" int settles(float x, float y, float a, float b) {\n'
                   '    return jr::settles(x, y, a, b); }\n')
    lib = str(d / "s.so")
    subprocess.run(["g++", "-O2", "-ffp-contract=off", "-shared", "-fPIC", "-I", CSRC, str(src),
                    "-o", lib], check=True)
    fn = ctypes.CDLL(lib).settles
    return lambda z, c: bool(fn(*(ctypes.c_float(v) for v in (z.real, z.imag, c.real, c.imag))))


def test_settled_orbits_never_escape(settles):
    """Orbits of 0 after some steps, and points up to the rims of the discs about
    cycles of period 1 and 2, for constants in and outside the first two bulbs."""
    rng = np.random.default_rng(3)
    settled = tried = 0
    for _ in range(4000):
        c = complex(rng.uniform(-1.4, 0.5), rng.uniform(-0.8, 0.8))
        root = cmath.sqrt(1 - 4 * c) if rng.random() < 0.6 else cmath.sqrt(-3 - 4 * c)
        z = (1 - root) / 2 if rng.random() < 0.6 else (-1 + root) / 2
        if rng.random() < 0.3:
            z = 0j
            for _ in range(int(rng.integers(0, 200))):
                z = z * z + c if abs(z) < 2 else z
        else:
            a, d = rng.uniform(0, 2 * math.pi), 10 ** rng.uniform(-4, 0)
            z += d * complex(math.cos(a), math.sin(a))
        if not settles(z, c):
            continue
        settled += 1
        for dt in ("fp32", "fp64", "ff"):
            n = 300 if dt == "ff" else 1500
            assert oracle.count(z, c, n, dt) == n, (z, c, dt)
    assert settled > 300


def test_what_does_not_settle(settles):
    """Repelling and parabolic points, escaping orbits, NaN and infinities."""
    for z, c in ((0j, 1j), (0.5 + 0j, 0.25 + 0j), (2 + 0j, -2 + 0j), (1.9 + 0j, 0j), (1 + 0j, 0j),
                 (complex(math.nan, 0), 0j), (complex(math.inf, 0), 0j), (0j, complex(0, math.nan)),
                 (complex(1e30, 1e30), 0j), (0j, 0.3 + 0.6j)):
        assert not settles(z, c)
    assert settles(0j, 0j) and settles(-1 + 0j, -1 + 0j) and settles(0j, -1 + 0.1j)
