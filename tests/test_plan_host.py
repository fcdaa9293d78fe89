"""The plan code behind the C ABI (buffers, streams, captures, choice of the form) on the host: the built
library over a HIP runtime that hands out addresses, runs no kernel and records every call
(host/fake_hip.hpp). Each scenario of host/plan_host_check.cpp is one test."""

import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
LIBDIR = os.path.join(os.path.dirname(HERE), "paper_1507_05156_amd")
SCENARIOS = ("captured_buffers_stay", "growth_frees", "streams_in_order", "threads_one_at_a_time",
             "captures_without_plan_memory", "first_sum_allocates_once", "tuned_call_without_room",
             "symmetry_switch", "same_kernel_for_a_k_range", "captures_use_what_is_there", "fp32_captures_use_what_is_there",
             "fused_sums_beyond_the_cap", "refused_sum_is_not_profiled", "batched_route",
             "wait_limit_runs_the_split_form", "grid_forms_of_the_device_tests",
             "device_nearly_full")


@pytest.fixture(scope="module")
def check(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no host C++ compiler")
    if not os.path.exists(os.path.join(LIBDIR, "libfockmi.so")):
        pytest.skip("library not built")
    if not os.path.exists("/opt/rocm/include/hip/hip_runtime.h"):
        pytest.skip("no HIP headers")
    exe = str(tmp_path_factory.mktemp("plan") / "plan_host_check")
    subprocess.run([gxx, "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-rdynamic", "-w",
                    os.path.join(HERE, "host", "plan_host_check.cpp"), "-L", LIBDIR, "-lfockmi", "-lpthread",
                    f"-Wl,-rpath,{LIBDIR}", "-Wl,--allow-shlib-undefined", "-o", exe], check=True)
    return exe


def test_scenarios_listed(check):
    listed = subprocess.run([check], check=True, capture_output=True, text=True).stdout.split()
    assert sorted(listed) == sorted(SCENARIOS)


@pytest.mark.parametrize("name", SCENARIOS)
def test_plan_code(check, name):
    env = {k: v for k, v in os.environ.items() if not k.startswith("FOCKMI_")}
    r = subprocess.run([check, name], capture_output=True, text=True, timeout=120, env=env)
    assert r.returncode == 0, r.stdout + r.stderr
