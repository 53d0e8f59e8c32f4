"""One-image calls: orbits ended in traps of every number of discs, views whose orbits
run long and so take the rows kernel, and grids of four waves a workgroup, against the
oracle on both sides of each rule."""
import time

import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
import paper_1611_03079_amd as jr  # noqa: E402

pytestmark = pytest.mark.gpu

# traps of periods 1, 2, 3, 4, 5, 7 (more than jr_small's discs from 5 on), none
TRAPPED = [0.1 + 0.1j, 0.2495 + 0j, -1 + 0.1j, -0.7495 + 0j, -0.1225 + 0.7449j, -1.3107 + 0j,
           0.282 + 0.53j, -0.504 + 0.563j, 0.3856 + 0.1428j, 0.3 + 0.6j]
SIEGEL, SEA = -0.390541 - 0.586788j, -0.7269 + 0.1889j


@pytest.mark.parametrize("dtype", ["fp64", "fp32", "ff"])
def test_images_with_traps_equal_the_oracle(dtype):
    pal = np.arange(201, dtype=np.uint32) * np.uint32(2654435)
    dev = torch.from_numpy(pal.view(np.int32).copy()).cuda()
    for c in TRAPPED:
        for win, w, h in (((-1.6, 1.6, -1.2, 1.2), 101, 67), ((-0.9, 0.6, -0.4, 0.7), 66, 45)):
            for cap in (129, 300):
                want = oracle.render(c, win, w, h, cap, dtype)
                got = jr.render(c, win, w, h, cap, dtype)
                col = jr.render(c, win, w, h, cap, dtype, palette=dev)
                torch.cuda.synchronize()
                np.testing.assert_array_equal(got.cpu().numpy(), want, err_msg=str((c, win, cap)))
                np.testing.assert_array_equal(col.cpu().numpy().view(np.uint32),
                                              oracle.colorize(want, pal))


def check(c, win, w, h, cap, dtype, mode="julia"):
    """The image, and its colours, at sampled pixels (all of one small row band too)."""
    out = torch.full((h, w), -1, dtype=torch.int32, device="cuda")
    got = jr.render(c, win, w, h, cap, dtype, out=out, mode=mode).cpu().numpy()
    assert got.min() >= 0 and got.max() <= cap
    rng = np.random.default_rng(w + h)
    n = 3000 if dtype == "ff" else 20000
    ii, jj = rng.integers(0, w, n).astype(np.int32), rng.integers(0, h, n).astype(np.int32)
    ii[:300], jj[:300] = np.arange(300) + w - 300, h - 1  # the last row's end
    ii[300:600], jj[300:600] = np.arange(300), 0
    want = oracle.render_pixels(c, win, w, h, cap, ii, jj, dtype, mode)
    np.testing.assert_array_equal(got[jj, ii], want, err_msg=str((c, win, w, h, cap, dtype, mode)))


PART = (0.1, 0.4, 0.09, 0.31)


@pytest.mark.parametrize("dtype", ["fp64", "fp32", "ff"])
@pytest.mark.parametrize("w, h", [(723, 725), (725, 725)])  # 524175 and 525625 pixels
def test_long_views_from_half_a_million_pixels(dtype, w, h):
    for cap in (128, 129):
        for c, win in ((SIEGEL, PART), (0.25 + 0j, PART), (1j, PART), (SIEGEL, (-1.6, 1.6, -1.2, 1.2)),
                       (2.5 + 0.1j, PART)):
            check(c, win, w, h, cap, dtype)
        for wd in (0.01, 0.9e-3, 1.1e-3):
            x, y = -0.743643887037151, 0.13182590420533
            check(0j, (x - wd / 2, x + wd / 2, y - wd / 2, y + wd / 2), w, h, cap, dtype,
                  "mandelbrot")


@pytest.mark.parametrize("dtype", ["fp64", "fp32"])
@pytest.mark.parametrize("w, h", [(2449, 2449), (2450, 2450)])  # about 6 million pixels
def test_long_views_from_six_million_pixels(dtype, w, h):
    for cap in (128, 200):
        check(SEA, PART, w, h, cap, dtype)
        check(0j, (-0.8, -0.7, 0.1, 0.2), w, h, cap, dtype, "mandelbrot")
        check(0j, (-2.1, 0.9, -1.2, 1.2), w, h, cap, dtype, "mandelbrot")


@pytest.mark.parametrize("dtype", ["fp64", "fp32", "ff"])
@pytest.mark.parametrize("w, h", [(2033, 1551), (2049, 2047), (17, 196613), (1, 262201), (4096, 1537)])
def test_workgroups_of_four_waves(dtype, w, h):
    """Grids of a little under and over 49152 waves, ragged at both edges."""
    for win in ((-1.6, 1.6, -1.2, 1.2), (-1.6, 1.5, -1.2, 1.25)):
        want = oracle.render(-0.4 + 0.6j, win, w, h, 9, dtype)
        out = torch.full((h, w), -1, dtype=torch.int32, device="cuda")
        got = jr.render(-0.4 + 0.6j, win, w, h, 9, dtype, out=out)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(got.cpu().numpy(), want)


def test_a_long_view_under_capture():
    out = torch.empty((725, 725), dtype=torch.int32, device="cuda")
    other = torch.empty_like(out)
    args = (SIEGEL, PART, 725, 725, 200, "fp32")
    want = jr.render(*args, out=other).clone()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        jr.render(*args, out=out)
    for _ in range(3):
        out.zero_()
        g.replay()
        jr.render(*args, out=other)
        torch.cuda.synchronize()
        assert torch.equal(out, want) and torch.equal(other, want)


def test_a_long_view_takes_no_longer_than_on_the_rows_kernel():
    """C = -0.3905 - 0.5868i, FP32, cap 1000, 1920x1080: 215 us; one thread per pixel 303."""
    rows = jr.Schedule(64, 2, 8, 0, 16, 0, 16, "cost", "rows", 16, 64)
    out = torch.empty((1080, 1920), dtype=torch.int32, device="cuda")

    def best(schedule):
        times = []
        for _ in range(10):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            for _ in range(10):
                jr.render(SIEGEL, PART, 1920, 1080, 1000, "fp32", out=out, schedule=schedule)
            torch.cuda.synchronize()
            times.append(time.perf_counter() - t0)
        return min(times)
    assert best(None) < 1.3 * best(rows)
