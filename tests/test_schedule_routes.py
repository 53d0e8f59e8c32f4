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


@pytest.mark.parametrize("dtype, cap, side, kept", [
    ("fp64", 128, 1024, True), ("ff", 100, 2000, True), ("fp32", 100, 2000, False),
    ("fp64", 129, 2000, False), ("ff", 100, 1023, False)])
def test_large_mandelbrot_images_of_low_caps_keep_it(monkeypatch, dtype, cap, side, kept):
    seen = []
    monkeypatch.setattr(jr, "tuned_schedule", lambda *a: PLAIN)
    monkeypatch.setattr(jr, "_out_tensor", lambda out, shape: torch.zeros(shape, dtype=torch.int32))
    monkeypatch.setattr(jr, "_stream_ptr", lambda s: ctypes.c_void_p(0))
    monkeypatch.setattr(jr, "_palette_ptr", lambda p: (ctypes.c_void_p(4), 2))
    monkeypatch.setattr(jr.lib, "julia_render_batch_colored",
                        lambda *a: seen.append(a[6]) or 0)
    for what in (dict(mode="mandelbrot"), dict(mode="mandelbrot", degree=3), dict(degree=4)):
        jr.render(0j, (-2, 1, -1, 1), side, side, cap, dtype, palette=object(), **what)
    assert [s is not None for s in seen] == [kept, False, False]


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


class Image:
    c, window, width, height, max_iter, dtype = 0.1j, (-1, 1, -1, 1), 40, 30, 90, "fp64"
    mode, degree, lam = "julia", 2, None

    def __init__(self, **kw):
        self.__dict__.update(kw)


@pytest.fixture
def table(monkeypatch):
    """A per-size table with a caller's entries and nothing else."""
    monkeypatch.setattr(jr, "_IMAGE_SCHEDULES_DONE", True)
    monkeypatch.setattr(jr, "_IMAGE_ENTRIES", {})
    jr.lib.jr_clear_image_schedules()
    mine = {("fp64", 128, 5000): ROWS, ("fp64", 90, 1200): jr.Schedule(64, 4, kernel="rows"),
            ("ff", 2 ** 31 - 1, 2 ** 63 - 1): jr.Schedule(16, 16)}
    for k, s in mine.items():
        jr.set_image_schedule(*k, s)
    yield mine
    jr.lib.jr_clear_image_schedules()


def test_timing_a_plain_entry_leaves_the_per_size_table(table):
    def timed():
        assert jr.image_schedule("fp64", 90, 1200) == PLAIN
        return 7.0
    assert autotune._as_image(Image(), PLAIN, timed) == 7.0
    assert jr.image_entries() == table
    for k, s in table.items():
        assert jr.image_schedule(*k) == s

    def fails():
        raise RuntimeError("x")
    with pytest.raises(RuntimeError):
        autotune._as_image(Image(), PLAIN, fails)
    assert jr.image_entries() == table
    # entries beyond the binding's knowledge are not brought back
    jr.lib.jr_clear_image_schedules()
    assert jr.image_entries() == {} and autotune._as_image(Image(), PLAIN, timed) == 7.0
    assert jr.image_entries() == {}


def test_timing_a_plain_entry_in_a_full_or_plain_table(table):
    for k in range(61):
        jr.set_image_schedule("fp32", 1000 + k, 100, ROWS)
    full = jr.image_entries()
    assert len(full) == 64

    def timed():
        return jr.image_schedule("fp64", 90, 1200).kernel
    assert autotune._as_image(Image(), PLAIN, timed) == "plain"
    assert jr.image_entries() == full
    jr.set_image_schedule("fp64", 90, 1200, PLAIN)  # already plain: nothing is touched
    full = jr.image_entries()
    assert autotune._as_image(Image(), PLAIN, lambda: jr.image_entries() == full) is True


@pytest.mark.parametrize("what", [dict(degree=3), dict(lam=0.01 + 0j)])
def test_a_general_map_s_plain_candidate_is_the_plain_kernel(monkeypatch, what):
    """Its one-image calls are batches of one and run what they are given."""
    seen = []
    monkeypatch.setattr(torch, "empty", lambda *a, **k: None)
    monkeypatch.setattr(torch.cuda, "synchronize", lambda: None)
    monkeypatch.setattr(jr, "render", lambda *a, **k: seen.append(k["schedule"]))
    autotune.time_render_wall(Image(**what), PLAIN, reps=1, calls=1)
    assert seen and all(s == PLAIN for s in seen)
    monkeypatch.setattr(autotune, "time_plan", lambda fr, s, **k: s.kernel)
    assert autotune.time_render_plain(Image(**what)) == "plain"


def test_the_shipped_cache_says_what_its_times_are():
    """Every entry carries a measured time; one chosen by hand says so, and what the
    time was taken on, and claims no search."""
    import json
    cache = json.load(open(autotune.os.path.join(autotune.os.path.dirname(autotune.__file__),
                                                 "autotune_cache.json")))
    entries = {k: e for k, e in cache.items() if k != "_workloads"}
    assert len(entries) >= 54
    for k, e in list(entries.items()) + list(cache["_workloads"].items()):
        assert e["ms"] > 0, k
        assert jr.check_schedule(jr.Schedule(**e["schedule"])) == jr.JR_OK
        if e.get("chosen") == "by hand":
            assert e["timed_on"] and "candidates" not in e, k
