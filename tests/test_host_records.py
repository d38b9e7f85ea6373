"""What calls that read results from pinned host records leave behind, on a HIP
runtime that queues kernels without running them (tests/host)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = "/opt/rocm/bin/hipcc"


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not installed")
    exe = str(tmp_path_factory.mktemp("stub") / "stub_runtime")
    p = subprocess.run([HIPCC, "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-x", "c++", os.path.join(ROOT, "tests", "host", "stub_runtime.cpp"),
                        "-rdynamic", "-ldl", "-o", exe], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True,
                       timeout=300)
    assert p.returncode == 0, p.stdout
    lib = os.path.join(ROOT, "paper_2409_17658_amd", "libmpr.so")
    return lambda mode: subprocess.run([exe, lib, mode], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True,
                                       timeout=120)


def test_failed_launch_leaves_no_writer_behind(driver):
    """A record goes back to the pool only when no queued kernel can write it,
    whichever launch of the call is reported as failed; and a failed
    allocation is not reported again by the next call."""
    p = driver("errors")
    assert p.returncode == 0, p.stdout


def test_synchronous_calls_return_with_the_stream_drained(driver):
    """mpr_find_period and mpr_sparse_plan_bytes are synchronous: the kernel
    that wrote the record a call waited for has retired when they return.
    A checked product has run as well: only its check, which runs behind it and
    wrote the record, may still be retiring."""
    p = driver("idle")
    assert p.returncode == 0, p.stdout


def test_long_waits_sleep(driver):
    """A call that waits for a record for 400 ms uses the processor for less than
    a quarter of them (the first 10 are spent looking)."""
    p = driver("wait")
    assert p.returncode == 0, p.stdout
