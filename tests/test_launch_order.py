"""The rules by which calls whose workgroups wait for one another follow each other from several streams (rt_launch_order.h), on the
CPU: the header is compiled with streams that are numbers (launch_order_check.cpp)."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2604_21215_amd", "csrc")


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("launch_order") / "check")
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-pthread", "-I", CSRC, os.path.join(HERE, "launch_order_check.cpp"), "-o", exe],
                   check=True)
    return exe


@pytest.mark.parametrize("check", ["rules", "captures", "owners_go", "threads"])
def test_launch_order(program, check):
    r = subprocess.run([program, check], stdout=subprocess.PIPE, text=True, timeout=30)
    assert r.returncode == 0, r.stdout
