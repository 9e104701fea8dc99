"""Failure handling and bookkeeping of the library's host code, without a GPU:
sonosim_api.cpp and sonosim_batch.cpp linked with a stand-in for the HIP
runtime and the kernel launchers (fake_hip.cpp), which records what is
enqueued and can make a launch fail."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(ROOT, "paper_2507_01152_amd", "csrc")


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("fake_hip") / "fake_hip")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-ffp-contract=off", "-w", "-D__HIP_PLATFORM_AMD__",
                    "-I/opt/rocm/include", "-I" + CSRC, "-I" + os.path.join(ROOT, "include"),
                    os.path.join(HERE, "fake_hip.cpp"), os.path.join(CSRC, "sonosim_api.cpp"),
                    os.path.join(CSRC, "sonosim_batch.cpp"), "-o", exe], check=True)

    def run(*args):
        r = subprocess.run([exe, *args], capture_output=True, text=True, timeout=120)
        assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-2000:]
    return run


def test_failed_step_leaves_nothing_behind(program):
    program("failed_step")


def test_tuner_skips_shapes_that_fail(program, tmp_path):
    program("failed_tuning", str(tmp_path / "tune.jsonl"))


def test_counters_are_clear_before_the_first_call(program):
    program("first_call")


def test_pinned_staging_is_allocated_once(program):
    program("staging")
