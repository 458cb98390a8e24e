"""The solve server's handling of failures and its bookkeeping, without a GPU:
csrc/server.cpp built with the host compiler against a HIP runtime that does,
or fails, everything at once (host/server_host.cpp)."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2207_11571_amd", "csrc")
ROCM_INCLUDE = "/opt/rocm/include"


def _build(exe, *flags):
    if not shutil.which("g++") or not os.path.isdir(os.path.join(ROCM_INCLUDE, "hip")):
        pytest.skip("no host compiler or no HIP headers")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-pthread", "-w", "-D__HIP_PLATFORM_AMD__", "-I", ROCM_INCLUDE,
                        "-I", CSRC, *flags, os.path.join(HERE, "host", "server_host.cpp"),
                        os.path.join(CSRC, "server.cpp"), "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return exe


@pytest.fixture(scope="module")
def server_host(tmp_path_factory):
    return _build(str(tmp_path_factory.mktemp("host") / "server_host"))


def _run(exe, scenario):
    r = subprocess.run([exe, scenario], capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stdout + r.stderr


@pytest.mark.parametrize("result", ["small", "large"])
def test_copy_that_fails_fails_the_solve(server_host, result):
    """A finished state that cannot be copied out whole is no result."""
    _run(server_host, f"copy_error_{result}")


def test_missing_streams_and_buffers_fail_the_creation(server_host):
    """A stream or a pinned buffer that cannot be had is an error of
    solve_server_create, not of the solves."""
    _run(server_host, "create_errors")


def test_copies_leave_the_null_stream_alone(server_host):
    _run(server_host, "null_stream")


@pytest.mark.parametrize("result", ["small", "large"])
def test_finished_solve_does_not_wait_for_the_next_round(server_host, result):
    """Its result is delivered and its slot free while the next round of its
    order is still being enqueued."""
    _run(server_host, f"delivery_{result}")


def test_failed_fallback_gives_its_block_away_when_nothing_writes_to_it(server_host):
    _run(server_host, "fallback_error")


@pytest.mark.parametrize("scenario", ["polling", "null_stream", "delivery_large", "copy_error_large",
                                      "fallback_error"])
def test_threads_of_the_server_do_not_race(tmp_path_factory, scenario):
    """The scenarios, and requests polled from the start, under the thread
    sanitizer."""
    exe = os.path.join(tmp_path_factory.getbasetemp(), "server_host_threads")
    if not os.path.exists(exe):
        _build(exe, "-g", "-fsanitize=thread")
    r = subprocess.run([exe, scenario], capture_output=True, text=True, timeout=100)
    if "FATAL: ThreadSanitizer" in r.stderr:
        pytest.skip("the thread sanitizer does not run on this kernel")
    assert r.returncode == 0, r.stdout + r.stderr
