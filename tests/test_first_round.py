"""The first round of the searches on the receive side, in lists of up to 2^31 - 1 values, without a GPU: no probe
outside the list, whatever the lane's number (32 probes of a list of 1,090,785,345 values and more: the lanes behind
them would wrap to positions before it), and the answer inside the bracket that the round leaves."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_probes_stay_inside_the_list(tmp_path):
    compiler = shutil.which("g++")
    if compiler is None:
        pytest.skip("no g++")
    exe = str(tmp_path / "first_round_host")
    subprocess.run([compiler, "-std=c++17", "-O1", "-Wall", "-Wextra", "-Werror", "-fsanitize=undefined",
                    "-fno-sanitize-recover=undefined", "-I", os.path.join(ROOT, "paper_1712_01887_amd", "csrc"),
                    os.path.join(ROOT, "tests", "first_round_host.cc"), "-o", exe], check=True, capture_output=True, text=True)
    run = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert run.returncode == 0 and run.stdout.startswith("ok "), run.stdout + run.stderr
