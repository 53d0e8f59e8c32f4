"""A call of one frame without a schedule runs the default of the frame's dtype, as a
call of several does."""
import numpy as np
import pytest

import oracle
from workloads import Frame

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_1611_03079_amd as jr  # noqa: E402

WIN = (-1.6, 1.6, -1.2, 1.2)
LAM = 0.002 + 0.001j


@pytest.mark.parametrize("dtype", ["fp64", "fp32", "ff"])
def test_one_frame_runs_the_default_schedule(dtype):
    """Tiles of the documented default (64 wide, lower for small launches), as a copy
    of it set by the caller gives too; the tiled stream took 16 x 16."""
    f = Frame(-0.8 + 0.156j, WIN, 131, 90, 100, dtype)
    want = oracle.render(f.c, f.window, f.width, f.height, f.max_iter, dtype)
    d = jr.default_schedule(dtype)
    for again in (False, True):
        if again:
            jr.set_default_schedule(dtype, d)
        plan = jr.Plan([f])
        assert plan.info()["tiles"] == 3 * 45
        plan.set_progress(torch.zeros(1, dtype=torch.int32, device="cuda"))  # the rows kernel
        plan.launch()
        torch.cuda.synchronize()
        np.testing.assert_array_equal(plan.views[0].cpu().numpy(), want)
        plan.close()


@pytest.mark.parametrize("degree, lam", [(2, None), (3, None), (8, None), (2, LAM), (3, LAM)])
def test_one_fp64_frame_by_every_call_equals_the_oracle(degree, lam):
    for win, w, h in ((WIN, 97, 61), ((-1.6, 1.5, -1.2, 1.25), 64, 33)):
        f = Frame(-0.2 + 0.1j, win, w, h, 150, "fp64", "julia", degree, lam)
        want = oracle.render(f.c, win, w, h, 150, "fp64", "julia", degree, lam)
        arena = torch.full((w * h,), -1, dtype=torch.int32, device="cuda")
        got = [jr.render_batch([f])[1][0], jr.render_batch_noalloc([f], arena)[0],
               jr.render(f.c, win, w, h, 150, "fp64", degree=degree, lam=lam)]
        pal = np.arange(151, dtype=np.int32)  # colours that are the counts
        got += [jr.render_batch([f], palette=torch.from_numpy(pal).cuda())[1][0]]
        torch.cuda.synchronize()
        for g in got:
            np.testing.assert_array_equal(g.cpu().numpy(), want)
        _, views = jr.render_batch([f], rows=[(5, h - 5)], arena=torch.full_like(arena, -1))
        torch.cuda.synchronize()
        band = views[0].cpu().numpy()
        np.testing.assert_array_equal(band[5:h - 5], want[5:h - 5])
        assert (band[:5] == -1).all() and (band[h - 5:] == -1).all()
