"""Host logic of the pipeline runner (csrc/run.cpp with csrc/stage.cpp), built with g++ under sanitizers on stand-ins for the
kernel launchers and the HIP runtime (tests/host/kernel_stubs.cpp, runtime_stubs.cpp).  Nothing in it can reach a GPU."""
import os
import subprocess

import pytest

from tests.test_host_sanitizers import build, run_clean

RUNNER = ["tests/host/kernel_stubs.cpp", "tests/host/runtime_stubs.cpp", "paper_2410_14312_amd/csrc/stage.cpp",
          "paper_2410_14312_amd/csrc/run.cpp"]


def test_an_order_that_cannot_be_satisfied_is_an_error(tmp_path_factory):
    run_clean(build(tmp_path_factory, "unsatisfiable_order", ["tests/host/unsatisfiable_order.cpp"] + RUNNER))


def test_runner_is_clean_under_sanitizers(tmp_path_factory):
    run_clean(build(tmp_path_factory, "sanitize_run", ["tests/host/sanitize_run.cpp", "paper_2410_14312_amd/csrc/schedule.cpp"] + RUNNER))


def test_issue_threads_do_not_race(tmp_path_factory):
    exe = build(tmp_path_factory, "race_run", ["tests/host/sanitize_run.cpp", "paper_2410_14312_amd/csrc/schedule.cpp"] + RUNNER, "thread")
    env = dict(os.environ)
    env.pop("LD_PRELOAD", None)
    r = subprocess.run([exe], capture_output=True, text=True, env=env, timeout=300)
    if "unexpected memory mapping" in r.stderr:
        pytest.skip("the thread sanitizer cannot map its shadow memory on this kernel")
    assert r.returncode == 0 and "WARNING" not in r.stderr, r.stderr[-2000:]
