"""One-image calls of small images, which run one thread per pixel with tests in
blocks (where escape is absorbing) and by half where the image is its own
rotation, against the oracle at the edges of the grid, of the blocks and of both
rules; and the frame records and views that the binding makes."""
import ctypes

import numpy as np
import pytest

import oracle
from workloads import Frame

torch = pytest.importorskip("torch")
import paper_1611_03079_amd as jr  # noqa: E402


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["fp64", "fp32", "ff"])
def test_small_images_equal_the_oracle(dtype):
    about0, off0 = (-1.6, 1.6, -1.2, 1.2), (-1.6, 1.5, -1.2, 1.25)
    for w, h in ((1, 1), (1, 2), (15, 3), (16, 4), (17, 5), (33, 8), (100, 100), (131, 77)):
        for cap in (0, 1, 7, 8, 9, 100):
            for c, win, mode in ((complex(-0.8, 0.156), about0, "julia"),
                                 (complex(-0.4, 0.6), off0, "julia"),
                                 (complex(-1.95, 0.1), about0, "julia"),
                                 (0j, (-1.2, 0.4, -0.9, 0.8), "mandelbrot"),
                                 (0j, (-2.2, 0.8, -1.2, 1.2), "mandelbrot")):
                if w * h > 200 and cap not in (9, 100):
                    continue
                got = jr.render(c, win, w, h, cap, dtype, mode=mode)
                torch.cuda.synchronize()
                want = oracle.render(c, win, w, h, cap, dtype, mode)
                np.testing.assert_array_equal(got.cpu().numpy(), want,
                                              err_msg="%s" % ((c, win, w, h, cap, mode),))


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["fp64", "fp32", "ff"])
def test_single_views_of_long_bounded_orbits(dtype):
    """Orbits that settle about cycles of period 1 and 2, or repeat, before the cap."""
    for win, c, mode, cap in (((-2.3, 0.9, -1.2, 1.25), 0j, "mandelbrot", 700),
                              ((-0.8, -0.7, -0.06, 0.07), 0j, "mandelbrot", 300),
                              ((-1.3, -1.2, -0.05, 0.06), 0j, "mandelbrot", 257),
                              ((-1.6, 1.6, -1.2, 1.2), -0.75 + 0j, "julia", 400)):
        got = jr.render(c, win, 90, 71, cap, dtype, mode=mode)
        torch.cuda.synchronize()
        want = oracle.render(c, win, 90, 71, cap, dtype, mode)
        assert (want == cap).sum() > 100
        np.testing.assert_array_equal(got.cpu().numpy(), want)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["fp64", "fp32", "ff"])
def test_narrow_tall_images(dtype):
    """More blocks of rows than a grid's 65535: each takes several."""
    for w, h, win in ((1, 300001, (-1.6, 1.5, -1.2, 1.25)), (17, 270003, (-1.6, 1.6, -1.2, 1.2))):
        got = jr.render(complex(-0.4, 0.6), win, w, h, 20, dtype)
        torch.cuda.synchronize()
        want = oracle.render(complex(-0.4, 0.6), win, w, h, 20, dtype)
        np.testing.assert_array_equal(got.cpu().numpy(), want)


@pytest.mark.gpu
def test_output_views():
    """Images land in the first elements of a larger tensor and of a slice."""
    c, win = complex(-0.8, 0.156), (-1.5, 1.5, -1.5, 1.5)
    want = oracle.render(c, win, 30, 20, 50, "fp64")
    big = torch.full((1000,), -1, dtype=torch.int32, device="cuda")
    for out in (big, big[100:], torch.empty((20, 30), dtype=torch.int32, device="cuda"),
                torch.empty(600, dtype=torch.int32, device="cuda")):
        got = jr.render(c, win, 30, 20, 50, "fp64", out=out)
        assert got.shape == (20, 30) and got.data_ptr() == out.data_ptr()
        np.testing.assert_array_equal(got.cpu().numpy(), want)
    assert (big[700:] == -1).all()
    frames = [Frame(c, win, 30, 20, 50, "fp64"), Frame(c, win, 7, 9, 50, "fp32")]
    arena, views = jr.render_batch(frames, arena=big[100:], offsets=[70, 3])
    torch.cuda.synchronize()
    for f, v, o in zip(frames, views, (70, 3)):
        assert v.data_ptr() == arena.data_ptr() + 4 * o and v.is_contiguous()
        np.testing.assert_array_equal(v.cpu().numpy(), oracle.render(
            f.c, f.window, f.width, f.height, f.max_iter, f.dtype))


def test_frame_records():
    """Records packed in one go equal those filled field by field, and what a
    field does not hold is taken or refused as ctypes does."""
    fr = [Frame(complex(0.1, -0.2), (-1, 1.5, -2, 2), 7, 9, 11, "ff"),
          Frame(0j, (-2, 1, -1, 1), 5, 4, 3, "fp32", "mandelbrot"),
          Frame(1j, (-1, 1, -1, 1), 5, 4, 3, "fp64", "julia", 4, complex(0.5, -0.25))]
    arr = jr._frames_array(fr, [5, 1 << 40, 7], [(0, 0), (1, 3), (2, 4)])
    for a, f, o, r in zip(arr, fr, (5, 1 << 40, 7), ((0, 0), (1, 3), (2, 4))):
        assert complex(a.c.re, a.c.im) == f.c
        assert (a.w.re_min, a.w.re_max, a.w.im_min, a.w.im_max) == f.window
        assert (a.width, a.height, a.max_iter, a.dtype) == (f.width, f.height, f.max_iter,
                                                            jr.DTYPES[f.dtype])
        assert (a.mode, a.row_begin, a.row_end, a.degree) == (jr.MODES[f.mode], *r, f.degree)
        lam = f.lam or 0j
        assert (a.out_offset, a.map, a.reserved) == (o, int(f.lam is not None), 0)
        assert complex(a.lam.re, a.lam.im) == lam
    wide = Frame(0j, (-2, 1, -1, 1), 1 << 33, 4, 3, "fp32")
    assert jr._frames_array([wide], [0])[0].width == ctypes.c_int32(1 << 33).value
    with pytest.raises(TypeError):
        jr._frames_array([Frame(0j, (-2, 1, -1, 1), 2.5, 4, 3, "fp32")], [0])
