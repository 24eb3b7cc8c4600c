"""The rules by which rt_stack_prefill's side streams are lent (rt_side_streams.h), on the CPU: the header is compiled with streams
that are numbers (side_streams_check.cpp).  What a call waits for cannot be seen reliably on a device, whose hardware queues are
shared by streams that have nothing to do with each other."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2604_21215_amd", "csrc")


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("side_streams") / "check")
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-pthread", "-I", CSRC, os.path.join(HERE, "side_streams_check.cpp"), "-o", exe],
                   check=True)
    return exe


@pytest.mark.parametrize("check", ["unrelated_callers", "many_at_once", "threads"])
def test_side_streams(program, check):
    r = subprocess.run([program, check], stdout=subprocess.PIPE, text=True, timeout=30)
    assert r.returncode == 0, r.stdout
