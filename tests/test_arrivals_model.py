"""The words by which the workgroups of a one-launch build hand rows to each other, on the host: the device header compiled with
the host's compiler, its wavefronts as coroutines in many random orders (tests/arrivals_model.cpp)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_random_orders_of_the_hand_over(tmp_path):
    if not shutil.which("g++"):
        pytest.skip("no host compiler")
    exe = str(tmp_path / "model")
    subprocess.run(["g++", "-O1", "-std=c++17", "-D__device__=", "-D__forceinline__=inline", "-Wno-unknown-pragmas",
                    "-I" + os.path.join(ROOT, "paper_2406_17276_amd", "csrc"), os.path.join(ROOT, "tests", "arrivals_model.cpp"),
                    "-o", exe], check=True)
    run = subprocess.run([exe, "50000"], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=300)
    assert run.returncode == 0 and run.stdout.strip() == "ok 50000", run.stdout
