"""The second stream of a set of populations (csrc/pa_side_stream.hpp), compiled for
the CPU on a stand-in machine of two devices: its stream and events are made on the
device of the set's stream, also where another one is current, and the current device
stays the caller's.  It is used where what it hides exceeds what it costs."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1711_02146_amd", "csrc")


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("side")
    (d / "hip").mkdir()
    (d / "hip" / "hip_runtime.h").write_text("#pragma once\n")  # the calls are in the program
    exe = str(d / "side_stream_ref")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", f"-I{d}", "-I" + CSRC,
                           os.path.join(HERE, "side_stream_ref.cpp"), "-o", exe])
    return exe


@pytest.mark.parametrize("current,stream_dev", [(0, 0), (0, 1), (1, 0), (1, 1)])
def test_side_stream_is_on_the_sets_device(program, current, stream_dev):
    out = subprocess.check_output([program, str(current), str(stream_dev)], text=True)
    err, own, beside, elsewhere, ordered, now = (int(v) for v in out.split())
    assert err == 0
    # the group of work 10 on the set's stream, those of 5 and 3 beside it
    assert (own, beside, elsewhere, ordered) == (1, 2, 0, 1)
    assert now == current


# sites x tiles: 512 is L = 4 and 8192 L = 10 at 8 tiles, 1.6e6 L = 12 at 900
@pytest.mark.parametrize("sweeps,steps,work,two", [
    (1, 0, [512, 1728], False), (3, 0, [512, 1728], False), (10, 0, [512, 1728], True),
    (1, 0, [512, 1728, 8192], True), (1, 0, [100000, 1600000], True), (10, 0, [1600000], False),
    (1, 4, [512, 1728], False), (10, 4, [512, 1728], False), (10, 50, [512, 1728], True),
    (1, 50, [512, 1728], False)])
def test_second_stream_is_used_where_it_pays(program, sweeps, steps, work, two):
    out = subprocess.check_output([program, "0", "0", str(sweeps), str(steps), *map(str, work)],
                                  text=True)
    err, own, beside, elsewhere, ordered, now = (int(v) for v in out.split())
    assert (err, elsewhere, ordered, now) == (0, 0, 1, 0)
    assert own + beside == len(work) and (beside > 0) == two
