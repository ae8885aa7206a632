"""The pool of device buffers (tc2_memory.hip) as a host program over a model
of the device's memory (tests/c/memory_shim.cpp): several threads at once and
allocations that fail, without a GPU."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SHIM = os.path.join(ROOT, "tests", "c", "memory_shim.cpp")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


@pytest.fixture(scope="module")
def shim(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("memory") / "memory_shim")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-D__HIP_PLATFORM_AMD__",
                        f"-I{ROCM}/include", "-o", exe, "-x", "c++", SHIM, "-pthread"],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr

    def run(scenario):
        r = subprocess.run([exe, scenario], capture_output=True, text=True, timeout=60)
        assert r.returncode == 0 and r.stdout == "ok\n", r.stderr
    return run


def test_a_range_is_handed_on_only_when_its_chunks_are_unmapped(shim):
    shim("release_beside_grow")


def test_threads_grow_and_release(shim):
    shim("many_threads")


def test_releases_wait_and_leave_captures_of_other_threads_alone(shim):
    shim("release_beside_capture")


def test_released_buffers_of_a_scope_are_bounded_and_given_back(shim):
    shim("scope_under_pressure")


def test_streams_pass_between_calls(shim):
    shim("service_streams")


def test_trim_without_host_memory(shim):
    shim("trim_without_host_memory")
