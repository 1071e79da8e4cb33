"""The push queue's protocol (csrc/turn_queue.hpp) with threads as waves, one
of which reads the queue's count late: see native/turn_queue_check.cpp."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    out = tmp_path_factory.mktemp("turn_queue") / "check"
    subprocess.run(["g++", "-O1", "-std=c++17", "-pthread", "-o", str(out),
                    os.path.join(HERE, "native", "turn_queue_check.cpp")], check=True)
    return str(out)


def test_every_wave_empties_at_the_same_turns(program):
    r = subprocess.run([program, "helper"], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout


def test_a_count_read_behind_one_barrier_is_caught(program):
    r = subprocess.run([program, "late_read"], capture_output=True, text=True, timeout=120)
    assert r.returncode == 1, r.stdout
