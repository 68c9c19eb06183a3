"""The serving scheduler over two compute queues that finish in either order and
a download queue beside the uploads (tests/native/sched_two_queues.cpp), built
with AddressSanitizer and UndefinedBehaviorSanitizer; and the worker's wait
between two looks."""
import os
import shutil
import subprocess

import pytest

SRC = os.path.join(os.path.dirname(os.path.abspath(__file__)), "native", "sched_two_queues.cpp")


def test_two_queue_scenarios(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ is not available")
    out = str(tmp_path / "sched_two_queues")
    r = subprocess.run([gxx, "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined",
                        "-fno-sanitize-recover=undefined", "-pthread", SRC, "-o", out], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([out], capture_output=True, text=True, timeout=300)
    print(r.stdout)
    assert r.returncode == 0, r.stdout + r.stderr
    assert "all scenarios passed" in r.stdout
