"""Host logic of the pipeline runner (csrc/run.cpp with csrc/stage.cpp), built with g++ under sanitizers on stand-ins for the
kernel launchers and the HIP runtime (tests/host/kernel_stubs.cpp, runtime_stubs.cpp).  Nothing in it can reach a GPU."""
from tests.test_host_sanitizers import build, run_clean

RUNNER = ["tests/host/kernel_stubs.cpp", "tests/host/runtime_stubs.cpp", "paper_2410_14312_amd/csrc/stage.cpp",
          "paper_2410_14312_amd/csrc/run.cpp"]


def test_an_order_that_cannot_be_satisfied_is_an_error(tmp_path_factory):
    run_clean(build(tmp_path_factory, "unsatisfiable_order", ["tests/host/unsatisfiable_order.cpp"] + RUNNER))


def test_runner_is_clean_under_sanitizers(tmp_path_factory):
    run_clean(build(tmp_path_factory, "sanitize_run", ["tests/host/sanitize_run.cpp", "paper_2410_14312_amd/csrc/schedule.cpp"] + RUNNER))
