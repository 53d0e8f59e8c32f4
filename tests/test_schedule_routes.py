"""Which schedules the binding and the autotuner hand to the library.  In a cache
entry of one image "plain" names the single-image kernel; in a batch it names the
kernel that tests every iteration, so such an entry must not reach a batch call."""
import ctypes
from dataclasses import asdict

import pytest

torch = pytest.importorskip("torch")
import paper_1611_03079_amd as jr  # noqa: E402
from paper_1611_03079_amd import autotune  # noqa: E402

PLAIN = jr.Schedule(kernel="plain")
ROWS = jr.Schedule(64, 8, 8, 0, 8, 0, 16, "cost", "rows", 8, 0)


def entry(s):
    return {"schedule": asdict(s), "ms": 1.0}


@pytest.mark.parametrize("tuned, want", [(PLAIN, None), (ROWS, ROWS), (None, None)])
@pytest.mark.parametrize("what", [dict(mode="mandelbrot"), dict(degree=3), dict(lam=0.01 + 0j)])
def test_coloured_batches_of_one_take_no_plain_entry(monkeypatch, tuned, want, what):
    seen = []

    def call(arr, n, pal, plen, out, cap, sched, stream):
        seen.append(None if sched is None else jr.Schedule.from_c(sched._obj))
        return 0
    monkeypatch.setattr(jr, "tuned_schedule", lambda *a: tuned)
    monkeypatch.setattr(jr, "_out_tensor", lambda out, shape: torch.zeros(shape, dtype=torch.int32))
    monkeypatch.setattr(jr, "_stream_ptr", lambda s: ctypes.c_void_p(0))
    monkeypatch.setattr(jr, "_palette_ptr", lambda p: (ctypes.c_void_p(4), 2))
    monkeypatch.setattr(jr.lib, "julia_render_batch_colored", call)
    jr.render(0j, (-2, 1, -1, 1), 8, 6, 100, "fp64", palette=object(), **what)
    assert seen == [want]
    jr.render(0j, (-2, 1, -1, 1), 8, 6, 100, "fp64", palette=object(), plain=True, **what)
    assert seen[1].kernel == "plain"  # where it is asked for


def test_apply_cache_sets_batch_schedules(monkeypatch):
    monkeypatch.setattr(autotune, "device_name", lambda: "gfx950")
    got = {}
    monkeypatch.setattr(jr, "set_default_schedule", lambda dt, s: got.__setitem__(dt, s))
    key = lambda dt, **k: autotune.cache_key("gfx950", dt, 100, 1 << 24, **k)  # noqa: E731
    batch = jr.Schedule(64, 4, 8, 0, 8, 0, 16, "table", "rows", 8, 0)
    plain_batch = jr.Schedule(kernel="plain", order="table")
    autotune.apply_cache({key("fp64"): entry(PLAIN), key("fp32"): entry(ROWS),
                          key("ff"): entry(ROWS), key("ff", batch=True): entry(batch)})
    assert got == {"fp32": ROWS, "ff": batch}
    got.clear()
    autotune.apply_cache({key("fp32", batch=True): entry(plain_batch)})  # a batch's own winner
    assert got == {"fp32": plain_batch}
