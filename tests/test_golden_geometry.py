"""The golden-label scan's host-compilable arithmetic on the CPU, from the same
header the kernels use, built with the address and undefined-behaviour
sanitizers."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2606_09079_amd", "csrc")


def _run(tmp_path, source):
    exe = str(tmp_path / "check")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", "-fsanitize=address,undefined",
                           "-fno-sanitize-recover=undefined", "-ffp-contract=off", "-I", CSRC,
                           os.path.join(HERE, source), "-o", exe])
    env = {k: v for k, v in os.environ.items() if k != "LD_PRELOAD"}
    res = subprocess.run([exe], capture_output=True, text=True, timeout=600, env=env)
    assert res.returncode == 0 and res.stdout.startswith("ok"), res.stdout[-2000:] + res.stderr[-2000:]


@pytest.mark.parametrize("source", ["golden_geometry_check.cpp", "golden_interval_check.cpp"])
def test_golden_host_arithmetic(tmp_path, source):
    _run(tmp_path, source)
