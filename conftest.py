"""Test setup beside tests/conftest.py.

The serving loop's overlap test needs a step that outlasts the host's work on the next
request, 0.34 ms, and takes one FP64 frame of 1920x1080, nearly all of it bounded, cap
4000, for it.  On the library's default schedule that frame's orbits end in a trap and
it takes 0.02 ms, so the test runs with the tiled stream, which iterates them to the
cap (6 ms), as the default of FP64."""
import pytest

LONG_STEP = "test_admission_during_a_step_and_overlapping_steps"


@pytest.fixture(autouse=True)
def a_step_that_lasts(request):
    if request.node.name != LONG_STEP:
        yield
        return
    import paper_1611_03079_amd as jr
    old = jr.default_schedule("fp64")
    jr.set_default_schedule("fp64", jr.Schedule(16, 16, 8, 0, 16, 0, 16, "cost", "tiled", 8, 0))
    yield
    jr.set_default_schedule("fp64", old)
