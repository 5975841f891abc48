"""Host paths of the library on a device that is the host.

`tests/host/host_paths_check.cpp` is compiled with the library's host sources
against `tests/host/fake_device.h`, in which device memory is host memory, a
launch leaves a line in a log, and any call can be made to fail.  So the order of
launches, waits and copies, and what happens when one of them fails, are checked
on the CPU.
"""
import os
import re
import shutil
import subprocess

import pytest

from paper_1806_08815_amd import build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIP_INCLUDE = "/opt/rocm/include"


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None or not os.path.exists(os.path.join(HIP_INCLUDE, "hip", "hip_runtime_api.h")):
        pytest.skip("g++ or the HIP headers not found")
    csrc = os.path.join(ROOT, "paper_1806_08815_amd", "csrc")
    exe = str(tmp_path_factory.mktemp("host") / "host_paths_check")
    b = subprocess.run([gxx, "-O1", "-g", "-std=c++17", "-D__HIP_PLATFORM_AMD__",
                        '-DDAPT_BUILD_ID="host"', "-I", HIP_INCLUDE,
                        "-I", os.path.join(ROOT, "include"), "-I", csrc,
                        os.path.join(ROOT, "tests", "host", "host_paths_check.cpp"),
                        os.path.join(csrc, "da_tables.cpp"), "-lpthread", "-o", exe],
                       capture_output=True, text=True, timeout=600)
    assert b.returncode == 0, b.stderr[-4000:]
    return exe


@pytest.mark.parametrize("check", [
    "batch_error",     # a failed launch of a batch: nothing is still running at the return
    "batch_overlap",   # both kernels' jobs of a batch side by side, no wait between
    "batch_chunks",    # more items than the tables hold
    "batch_stats",     # the launch shapes reported after a batch
    "create_waits",    # an instance made beside running anneals
    "create_memory",   # and with little device memory left
    "create_sizes",    # small ones are derived on the host
    "outputs_memory",  # large outputs to the host: device memory they take
    "outputs_pinned",  # small ones: without pinned memory, and a failed wait
    "error_once",      # a failed call's error does not reach the next call
    "server_tables",   # where a served job's tables are built
    "temps_bounded",   # the cache of temperature lists
    "tuner_windows",   # the launches that time the table-driven kernel's shapes
])
def test_host_path(program, check):
    r = subprocess.run([program, check], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout[-4000:] + r.stderr[-2000:]
    assert "failures 0" in r.stdout


def test_compiled_step_kernels_are_those_chosen(program):
    """Every variant of the wave and team kernels that the library holds is one that
    a launch shape asks for, and the other way round."""
    r = subprocess.run([program, "list_shapes"], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout[-2000:]
    chosen = {l for l in r.stdout.splitlines() if l.startswith(("wave", "team"))}
    if not os.path.exists(build.LIB):
        build.build_library()
    with open(build.LIB, "rb") as f:
        names = f.read()
    built = set()
    for m in re.finditer(rb"6k_waveI([asi])Li(\d+)ELb([01])ELb[01]ELb[01]E", names):
        built.add("wave %s %s %s" % tuple(g.decode() for g in m.groups()))
    for m in re.finditer(rb"6k_teamI([asi])Li(\d+)ELi(\d+)ELi(\d+)ELb[01]ELb[01]E", names):
        built.add("team %s %s %s %s" % tuple(g.decode() for g in m.groups()))
    assert chosen == built, (sorted(built - chosen), sorted(chosen - built))
