"""The stage executor's paths that launch several layers' work together, in a host-only sanitizer build (tests/host/joint_launches.cpp)."""
from tests.test_host_sanitizers import build, run_clean


def test_launches_of_several_layers_touch_their_own(tmp_path_factory):
    run_clean(build(tmp_path_factory, "joint_launches", ["tests/host/joint_launches.cpp", "tests/host/kernel_stubs.cpp", "paper_2410_14312_amd/csrc/stage.cpp",
                                                         "paper_2410_14312_amd/csrc/schedule.cpp"]))
