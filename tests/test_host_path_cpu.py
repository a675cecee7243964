"""The library's host path without a GPU: which kernels and graphs its calls launch (tests/fake_hip.py)."""

import os

import pytest

from tests.fake_hip import run


@pytest.fixture(scope="module", autouse=True)
def built():
    from paper_2205_04979_amd import depo
    if not os.path.exists(depo.library_path()):
        from paper_2205_04979_amd.build import build
        build()


@pytest.mark.parametrize("graph", [True, False])
@pytest.mark.parametrize("sizes,reorder", [([300], 0), ([300], 3), ([9000], 0), ([9000, 40], 16), ([0, 70], 0)])
def test_calls_run_the_steps_they_are_asked_for(tmp_path, sizes, reorder, graph):
    got = run(tmp_path, f"""
s = simulation({sizes}, reorder={reorder}, cfg=(1, 4, 64, 2), graph={graph})
out = []
total = 0
for n in (1, 15, 16, 17, 3, 130, 21, 64, 7):
    fake.fake_reset()
    assert s.step(n) == 0
    total += n
    out.append([n, steps_run(), s.steps_done() - total])
print(json.dumps(out))
""")
    assert all(asked == done and off == 0 for asked, done, off in got), got


@pytest.mark.parametrize("calls,failing", [((17,), 0), ((17,), 1), ((5, 130), 1), ((20, 3), 1), ((20, 130, 3), 1)])
def test_a_failed_capture_leaves_host_and_device_at_the_same_step(tmp_path, calls, failing):
    """A call whose graph cannot be captured returns an error; the steps that the host counts are those that
    ran, so that the next call goes on from there."""
    got = run(tmp_path, f"""
s = simulation([9000])
fake.fake_reset()
fake.fake_fail_capture({failing})
status = [s.step(n) for n in {calls}]
print(json.dumps(dict(status=status, ran=steps_run(), counted=s.steps_done())))
""")
    assert got["ran"] == got["counted"], got
