"""Images that equal their own 180-degree rotation: an even map on a window
about 0.  The rows kernel computes half of such an image's rows and stores
each count at the opposite pixel too; the rest of the frames it computes whole.

On the CPU: the oracle's images of every form that the rule accepts have that
symmetry, and those it refuses need not.  On the GPU: the images equal the
oracle's, at the sizes where half an image can go wrong."""
import numpy as np
import pytest

import oracle
from workloads import Frame

C = complex(-0.72, 0.21)
LAM = complex(-0.02, 0.011)


def image(f, w=None, h=None):
    return oracle.render(f.c, f.window, w or f.width, h or f.height, f.max_iter, f.dtype, f.mode,
                         f.degree, f.lam)


EVEN = [Frame(c, (-rx, rx, -ry, ry), 0, 0, cap, dt, "julia", deg, lam)
        for deg in (2, 4, 6, 8) for dt in ("fp64", "fp32", "ff") for lam in (None, LAM)
        if not (lam and dt == "ff")
        for c, rx, ry, cap in ((C, 1.6, 1.2, 60), (complex(0.31, 0.0), 1.1, 1.7, 37))]


@pytest.mark.parametrize("size", [(1, 2), (7, 5), (16, 9), (33, 20)])
@pytest.mark.parametrize("k", range(len(EVEN)))
def test_even_maps_about_zero_are_their_own_rotation(k, size):
    img = image(EVEN[k], *size)
    np.testing.assert_array_equal(img, img[::-1, ::-1])


def test_the_oracle_tells_the_refused_forms_apart():
    """An odd degree, a window off 0 and a Mandelbrot image lack the symmetry."""
    for f in (Frame(C, (-1.6, 1.6, -1.2, 1.2), 33, 20, 60, "fp64", "julia", 3),
              Frame(C, (-1.6, 1.61, -1.2, 1.2), 33, 20, 60, "fp64"),
              Frame(C, (-1.6, 1.6, -1.2, 1.2001), 33, 20, 60, "fp64"),
              Frame(0j, (-1.6, 1.6, -1.2, 1.2), 33, 20, 60, "fp64", "mandelbrot")):
        img = image(f)
        assert (img != img[::-1, ::-1]).any(), f


SIZES = [(1, 1), (1, 2), (2, 1), (63, 3), (64, 4), (65, 5), (130, 67), (128, 64), (200, 129)]


@pytest.mark.gpu
@pytest.mark.parametrize("tile_h", [1, 2, 7, 16, 64])
@pytest.mark.parametrize("persistent", [0, 1])
def test_mirrored_images_equal_the_oracle(tile_h, persistent):
    """Odd and even sizes in every dtype, even degrees and the rational map
    beside frames that are not mirrored, whole and as bands of rows (only a
    band about the middle is mirrored), with colours and with counters."""
    import torch
    import paper_1611_03079_amd as jr
    frames, rows = [], []
    for k, (w, h) in enumerate(SIZES):
        dt = ("fp32", "fp64", "ff")[k % 3]
        frames.append(Frame(C, (-1.6, 1.6, -1.2, 1.2), w, h, 90, dt))
        frames.append(Frame(C, (-1.3, 1.3, -1.2, 1.2), w, h, 50, "fp32", "julia", 4))
        frames.append(Frame(C, (-1.3, 1.3, -1.2, 1.2), w, h, 40, "fp64", "julia", 2, LAM))
        frames.append(Frame(C, (-1.3, 1.3, -1.2, 1.2), w, h, 40, "fp64", "julia", 3))
        frames.append(Frame(C, (-1.3, 1.4, -1.2, 1.2), w, h, 40, "fp32"))
        frames.append(Frame(complex(1.7, 1.2), (-1.3, 1.3, -1.2, 1.2), w, h, 40, dt))
    for sub in (frames, [f for f in frames if f.dtype == "fp32" and f.degree == 2]):
        want = [image(f) for f in sub]
        sched = jr.Schedule(64, tile_h, 8, 0, 16, persistent, 16, "cost", "rows", 8, 24)
        plan = jr.Plan(sub, sched)
        done = torch.zeros(len(sub), dtype=torch.int32, device="cuda")
        plan.launch()
        torch.cuda.synchronize()
        for k, f in enumerate(sub):
            np.testing.assert_array_equal(plan.views[k].cpu().numpy(), want[k], err_msg=str(f))
        plan.arena.fill_(-1)
        plan.set_progress(done)
        plan.launch()
        torch.cuda.synchronize()
        assert done.cpu().tolist() == [f.pixels for f in sub]
        for k, f in enumerate(sub):
            np.testing.assert_array_equal(plan.views[k].cpu().numpy(), want[k], err_msg=str(f))
        plan.close()
        # bands of rows: about the middle, and one row off it
        for off in (0, 1):
            some = [k for k, f in enumerate(sub) if f.height > 4]
            bands = [(1 + off, sub[k].height - 1) for k in some]
            offs = [0] * len(some)
            for j in range(1, len(some)):
                offs[j] = offs[j - 1] + sub[some[j - 1]].pixels
            arena = torch.full((sum(sub[k].pixels for k in some),), -1, dtype=torch.int32,
                               device="cuda")
            _, views = jr.render_batch([sub[k] for k in some], sched, arena=arena, offsets=offs,
                                       rows=bands)
            torch.cuda.synchronize()
            for (a, b), k, v in zip(bands, some, views):
                got = v.cpu().numpy()
                np.testing.assert_array_equal(got[a:b], want[k][a:b], err_msg=str(sub[k]))
                assert (got[:a] == -1).all() and (got[b:] == -1).all()
        pal = np.arange(61, dtype=np.uint32) * np.uint32(2654435)
        _, views = jr.render_batch(sub, sched,
                                   palette=torch.from_numpy(pal.view(np.int32).copy()).cuda())
        torch.cuda.synchronize()
        for k, v in enumerate(views):
            np.testing.assert_array_equal(v.cpu().numpy().view(np.uint32),
                                          oracle.colorize(want[k], pal), err_msg=str(sub[k]))


@pytest.mark.gpu
def test_mirrored_cardioid_path_equals_the_oracle():
    import torch
    import paper_1611_03079_amd as jr
    import workloads as wl
    g = wl.growing_cardioid_path(6, 12, 3.9, 3.6, 75, 41, 80, "fp32")
    path = jr.CardioidPath(g.step, g.a0, g.da, g.window, g.frames, g.width, g.height, g.max_iter,
                           g.dtype)
    for sched in (None, jr.Schedule(64, 16, 8, 0, 16, 0, 16, "cost", "rows", 32, 64)):
        _, views = jr.render_cardioid_path(path, sched)
        torch.cuda.synchronize()
        for k, v in enumerate(views):
            c = oracle.cardioid_constant(g.step, g.a0, g.da, k)
            f = Frame(c, g.window, g.width, g.height, g.max_iter, g.dtype)
            np.testing.assert_array_equal(v.cpu().numpy(), image(f), err_msg="frame %d" % k)
