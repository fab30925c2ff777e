"""The pools behind the list and result copies (csrc/layout.cpp), compiled for
the host against a stand-in for the HIP runtime that keeps what is launched on a
stream until it is told to run it (tests/host/list_copies.cpp)."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1301_3494_amd", "csrc")


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("list_copies") / "list_copies")
    subprocess.run(["g++", "-std=c++17", "-O1", "-pthread", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    os.path.join(HERE, "host", "list_copies.cpp"), os.path.join(CSRC, "layout.cpp"), "-o", exe],
                   check=True)
    return exe


def run(program, check):
    r = subprocess.run([program, check], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr


@pytest.mark.parametrize("check", ["per_thread_streams", "ordinary_streams"])
def test_blocks_are_reused_in_stream_order_only(program, check):
    run(program, check)


def test_a_copy_that_was_not_launched_is_an_error(program):
    run(program, "failed_copies")


def test_host_arrays_are_free_once_a_list_is_on_its_way(program):
    run(program, "host_arrays_are_free")


@pytest.mark.parametrize("check", ["dead_streams", "list_memory", "pinned_sizes"])
def test_idle_blocks_are_given_back(program, check):
    run(program, check)
