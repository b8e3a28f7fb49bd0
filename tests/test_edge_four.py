"""The first and last loads of a part's pairs (warm-up densities, receive side), without a GPU: nothing behind a payload's
last pair and nothing before its first slot is read, and every pair arrives, wherever the part starts in a line."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_loads_stay_inside_the_payload(tmp_path):
    compiler = shutil.which("g++")
    if compiler is None:
        pytest.skip("no g++")
    exe = str(tmp_path / "edge_four_host")
    subprocess.run([compiler, "-std=c++17", "-O1", "-Wall", "-Wextra", "-Werror", "-I",
                    os.path.join(ROOT, "paper_1712_01887_amd", "csrc"), os.path.join(ROOT, "tests", "edge_four_host.cc"),
                    "-o", exe], check=True, capture_output=True, text=True)
    run = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert run.returncode == 0 and run.stdout.startswith("ok "), run.stdout + run.stderr
