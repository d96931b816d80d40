"""The library's launch rules, from the host alone: tests/launch_rules_check.cpp
is built against the library's internal headers and linked to liblqcd.so."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = "/opt/rocm/bin/hipcc"


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    if not os.path.exists(HIPCC):
        pytest.skip("no ROCm toolchain")
    from paper_2503_16994_amd import build
    if not os.path.exists(build.LIB):
        build.build()
    exe = str(tmp_path_factory.mktemp("rules") / "launch_rules_check")
    libdir = os.path.dirname(build.LIB)
    r = subprocess.run([HIPCC, "-x", "hip", "--offload-host-only", "-O1", "-std=c++17",
                        os.path.join(ROOT, "tests", "launch_rules_check.cpp"), "-x", "none", build.LIB,
                        f"-Wl,-rpath,{libdir}", "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
    return exe


@pytest.mark.parametrize("check", ["small_launches", "own_configurations", "converted_configurations", "tuning_round_trip",
                                   "workspace_bytes", "meson_scratch"])
def test_rule(program, check):
    r = subprocess.run([program, check], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-2000:]
