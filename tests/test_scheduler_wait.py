"""CPU: Scheduler::wait (csrc/scheduler.h) with an executor whose batches end
after a fixed time (tests/sched_wait.cpp), built with g++ plain and with the
undefined-behaviour, address and thread sanitizers."""
from __future__ import annotations

import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
INC = ["-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2404_01817_amd", "csrc")]
BUILDS = {"plain": ["-O2", "-Wall", "-Werror"],
          "undefined": ["-O1", "-fsanitize=undefined", "-fno-sanitize-recover=all"],
          "address": ["-O1", "-fsanitize=address"],
          "thread": ["-O1", "-fsanitize=thread"]}


@pytest.fixture(scope="module", params=sorted(BUILDS))
def program(request, tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("sched") / request.param)
    r = subprocess.run(["g++", "-std=c++17", "-g", "-pthread", *BUILDS[request.param], *INC,
                        os.path.join(ROOT, "tests", "sched_wait.cpp"), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return exe


@pytest.mark.parametrize("check", ["timeouts", "waiters", "destroyed"])
def test_wait(program, check):
    r = subprocess.run([program, check], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "checks passed" in r.stdout, r.stdout + r.stderr
    assert "Sanitizer" not in r.stderr, r.stderr
