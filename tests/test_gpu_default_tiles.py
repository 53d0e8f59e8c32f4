"""The library's default schedules lower their tiles for launches of few rows, which
tall tiles leave waiting for the slowest wave, and leave a caller's default alone."""
import numpy as np
import pytest

import oracle
from workloads import Frame

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_1611_03079_amd as jr  # noqa: E402

WIN = (-1.6, 1.5, -1.2, 1.25)


def frames(n, w, h, dtype, cap=100):
    return [Frame(complex(-0.7, 0.2 + 0.001 * k), WIN, w, h, cap, dtype) for k in range(n)]


# (frames, width, height) -> rows of a tile: 8192, 16320, 16384, 65280, 65536, 131072,
# 786240 and 788480 pairs of rows; the last holds ragged widths and an odd height
SHAPES = [((1, 1024, 1024), 2), ((2, 1024, 1020), 2), ((1, 1024, 2048), 4),
          ((2, 2048, 2040), 4), ((2, 2048, 2048), 8), ((1, 4096, 4096), 8),
          ((13, 3840, 2016), 8), ((14, 3520, 2048), 16), ((3, 67, 101), 2)]


@pytest.mark.parametrize("dtype", ["fp64", "fp32", "ff"])
def test_tiles_follow_the_size_of_the_launch(dtype):
    arena = torch.empty(14 * 3520 * 2048, dtype=torch.int32, device="cuda")
    for (n, w, h), rows in SHAPES:
        fr = frames(n, w, h, dtype) if n > 1 else frames(1, w, h // 2, dtype) * 2
        plan = jr.Plan(fr, arena=arena)
        h = fr[0].height
        assert plan.info()["tiles"] == len(fr) * -(-w // 64) * -(-h // rows), (n, w, h)
        plan.close()


@pytest.mark.parametrize("dtype", ["fp64", "fp32", "ff"])
def test_small_launches_equal_the_oracle_and_a_set_default_stays(dtype):
    fr = frames(3, 67, 101, dtype)
    want = [oracle.render(f.c, f.window, f.width, f.height, f.max_iter, dtype) for f in fr]
    old = jr.default_schedule(dtype)
    tall = jr.Schedule(64, 16, 8, 0, 24, 0, 16, "cost", "rows", 8, 0)
    for default in (old, tall):
        jr.set_default_schedule(dtype, default)
        try:
            plan = jr.Plan(fr)
            plan.launch()
            torch.cuda.synchronize()
            assert plan.info()["tiles"] == 3 * 2 * (51 if default == old else 7)
            for v, w in zip(plan.views, want):
                np.testing.assert_array_equal(v.cpu().numpy(), w)
            plan.close()
        finally:
            jr.set_default_schedule(dtype, old)
