"""Host code of the library (csrc/hs_host.cpp, hs_lib.cpp, hs_driver.cpp) compiled against a stand-in
for the HIP runtime (tests/host_double), on the CPU: what happens when memory or threads run out, and
how the waiting calls wait.  Every check runs in a process of its own."""
import os
import subprocess

import pytest

from paper_2402_04466_amd import build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HERE = os.path.join(ROOT, "tests", "host_double")


@pytest.fixture(scope="session")
def host_double(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("host_double") / "host_double")
    rocm = os.path.dirname(os.path.dirname(os.path.realpath(build.hipcc())))
    src = [os.path.join(build.CSRC, f) for f in ("hs_host.cpp", "hs_lib.cpp", "hs_driver.cpp")]
    src += [os.path.join(HERE, f) for f in ("fake_hip.cpp", "host_double_main.cpp")]
    subprocess.run([os.path.join(rocm, "llvm", "bin", "clang++"), "-std=c++17", "-O2", "-w",
                    "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(rocm, "include"), "-I",
                    os.path.join(ROOT, "include"), "-I", build.CSRC, *src, "-o", exe, "-lpthread", "-ldl"],
                   check=True)
    return exe


@pytest.mark.parametrize("check", ["packing_threads", "create_failures", "group_failures", "feed_failures",
                                   "call_failures", "mux_failures", "pinned_wait", "ready_result", "endless_wait",
                                   "prefetched_weights", "tile_grids", "one_queue_alone", "end_of_a_frame", "partition_failures", "callers_thread", "small_network_forms",
                                   "timed_small_network"])
def test_host_code(host_double, check):
    r = subprocess.run([host_double, check], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, (r.returncode, r.stdout[-500:], r.stderr[-500:])


@pytest.fixture(scope="session")
def plan(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("plan") / "plan")
    rocm = os.path.dirname(os.path.dirname(os.path.realpath(build.hipcc())))
    src = [os.path.join(HERE, "plan_main.cpp"), os.path.join(HERE, "fake_hip.cpp")]
    src += [os.path.join(build.CSRC, f) for f in ("hs_host.cpp", "hs_driver.cpp")]
    subprocess.run([os.path.join(rocm, "llvm", "bin", "clang++"), "-std=c++17", "-O2", "-w",
                    "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(rocm, "include"), "-I",
                    os.path.join(ROOT, "include"), "-I", build.CSRC, *src, "-o", exe, "-lpthread", "-ldl"],
                   check=True)
    return exe


def test_refused_plans(plan):
    r = subprocess.run([plan], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout[-500:]


def test_gpu_tests_run_every_convolution_kernel(plan):
    """The sizes of the GPU tests against the oracle take every kernel and form that the planner can choose."""
    import test_gpu_small_grids as t

    def forms(net, *tests):
        got = set()
        for test in tests:
            sizes = [m for m in test.pytestmark if m.name == "parametrize"][0].args[1]
            for size in sizes:
                r = subprocess.run([plan, net, *map(str, size)], capture_output=True, text=True, timeout=60)
                assert r.returncode == 0
                got |= set(r.stdout.split("\n")) - {""}
        return got
    big = forms("resnet18_convlstm", t.test_small_grid_convolutions_match_the_oracle,
                t.test_tiles_of_consecutive_pixels_match_the_oracle)
    assert big == {f"run {i}" for i in range(7)} | {f"s2_run {i}" for i in range(5)} | {"block64 0", "s2_dira 0"}, sorted(big)
    assert forms("tiny4", t.test_small_network_layers_match_the_oracle) == {"tiny_net 0"}


def test_tiles_of_consecutive_pixels(tmp_path):
    exe = str(tmp_path / "run_geometry")
    rocm = os.path.dirname(os.path.dirname(os.path.realpath(build.hipcc())))
    subprocess.run([os.path.join(rocm, "llvm", "bin", "clang++"), "-std=c++17", "-O2", "-w",
                    "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(rocm, "include"), "-I", build.CSRC,
                    os.path.join(HERE, "run_geometry_main.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout[-500:]
