"""The host code on a stand-in for the runtime (fake_hip.cpp: no GPU, kernels do nothing): calls that fail, and what is kept from
one call to the next."""
import os
import shutil
import subprocess

import pytest

from paper_1508_02363_amd import _lib

HERE = os.path.dirname(os.path.abspath(__file__))
EINVAL, ENOMEM, ENOCONV, EDEVICE = _lib.DBAR_EINVAL, _lib.DBAR_ENOMEM, _lib.DBAR_ENOCONV, _lib.DBAR_EDEVICE


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("no g++")
    exe = str(tmp_path_factory.mktemp("fake_hip") / "fake_hip")
    subprocess.run(["g++", "-O1", "-std=c++17", "-I" + os.path.join(os.path.dirname(HERE), "include"),
                    os.path.join(HERE, "fake_hip.cpp"), "-o", exe, "-rdynamic", "-ldl", "-pthread"], check=True)

    def call(scenario):
        r = subprocess.run([exe, _lib.LIB_PATH, scenario], capture_output=True, text=True, timeout=120)
        assert r.returncode == 0, r.stderr
        return [(a, int(b)) for a, b in (ln.split() for ln in r.stdout.splitlines())]

    return call


def test_an_error_left_by_the_caller_does_not_refuse_a_call(run):
    """(the stand-in's solve has nothing to converge to: DBAR_ENOCONV; the error is still there for its owner)"""
    assert run("left_error") == [("transform", 0), ("apply", 0), ("solve", ENOCONV), ("left", 101)]


def test_a_launch_that_fails_is_an_error(run):
    assert run("failed_launch") == [("k_stage_copy", EDEVICE), ("after", 0), ("k_lines", EDEVICE), ("after", 0),
                                    ("k_tail_table", EDEVICE), ("after", 0)]


def test_a_lost_read_of_the_flags_ends_the_solve(run):
    """The flags the host holds are then an earlier step's.  (Reads of a solve of 8 steps at N = 128: the start, every four
    steps, the cycle's end; at N = 64: the start, the cycle, its end.)"""
    solves = [b for a, b in run("lost_report") if a == "solve"]
    assert solves == 2 * [ENOCONV, EDEVICE, EDEVICE, EDEVICE]


def test_a_lost_read_of_the_flags_ends_the_requests_and_not_the_session(run):
    """The boxes, a cycle's flags, a cycle's end: the request ends with an error, the next one of its grid is served."""
    seen = run("lost_report_serving")
    assert [b for a, b in seen if a == "lost"] == [ENOCONV, EDEVICE, EDEVICE, EDEVICE]
    assert [b for a, b in seen if a == "next"] == 4 * [ENOCONV]
    assert seen[-1] == ("in_flight", 0)


def test_graphs_of_two_grids_of_one_size_are_kept(run):
    """Eight steps are two groups: two captures for each L, none when it comes back; a larger grid drops them (new buffers)."""
    assert [b for _, b in run("captures")] == [2, 4, 4, 4, 8]


def test_a_potential_with_nan_is_refused_as_such_and_first(run):
    """Also where there is no memory for its solve; nothing but the potential's own buffer is allocated before, and what an
    earlier solve captured is still there after."""
    seen = run("nan_first")
    assert [b for a, b in seen if a == "nan"] == 5 * [EINVAL]
    assert [b for a, b in seen if a == "memory"] == 2 * [ENOMEM]
    assert dict(seen)["most"] <= 16 * 1024 ** 2
    assert dict(seen)["captures"] == 0


def test_a_small_transform_waits_for_its_stream(run):
    """(one chunk; a wait for an event leaves the caller's next synchronisation of the device a slow one)"""
    assert run("transform_waits") == [("transform", 0), ("stream_waits", 1), ("transform", 0), ("stream_waits", 0)]


def test_the_timer_sees_every_launch(run):
    seen = dict(run("timer"))
    assert seen["made"] > 100 and seen["seen"] == seen["made"]
