"""Checks of the native library on the host, by a program that stands in for the HIP runtime (host_checks.cpp)."""

import os
import subprocess

import pytest

import paper_2411_15100_amd as xgm
from paper_2411_15100_amd import build as lib_build

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def host_checks(tmp_path_factory):
    xgm.load_library()  # (built if it is not)
    out = str(tmp_path_factory.mktemp("host_checks") / "host_checks")
    include = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "include")
    subprocess.run([os.environ.get("CXX", "g++"), "-O1", "-std=c++17", "-Wall", "-rdynamic", "-pthread", "-D__HIP_PLATFORM_AMD__", "-isystem", include,
                    os.path.join(HERE, "host_checks.cpp"), "-o", out, "-ldl"], check=True)

    def run(what):
        done = subprocess.run([out, lib_build.LIB, what], capture_output=True, text=True, timeout=120)
        assert done.returncode == 0, done.stdout + done.stderr

    return run


def test_a_build_ends_where_a_copy_cannot_be_launched(host_checks):
    host_checks("moves")


def test_copies_that_are_too_many_for_a_launch_are_refused(host_checks):
    host_checks("too_many_moves")
