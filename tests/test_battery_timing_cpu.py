"""Bookkeeping of the battery's timed launches, without a GPU: built from its
header with g++ and run against a simulated device whose clock runs on between
the host's questions."""

import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
SRC = os.path.join(HERE, "csrc", "timed_chain_check.cpp")
INC = os.path.join(os.path.dirname(HERE), "paper_1411_2484_amd", "csrc")


def test_no_event_is_given_back_while_a_launch_needs_it(tmp_path):
    exe = str(tmp_path / "timed_chain_check")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
                    "-I", INC, "-o", exe, SRC], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr
    assert r.stdout.strip() == "ok"
