"""The host's part of the per-layer procedure with a stand-in for the HIP runtime (tests/host_procedure_main.cpp): what it leaves behind when a step fails."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2605_14929_amd")


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("procedure") / "host_procedure")
    subprocess.check_call(["g++", "-std=c++17", "-g", "-O1", "-Wno-unused-result", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-rdynamic", "-o", exe,
                           os.path.join(ROOT, "tests", "host_procedure_main.cpp"), os.path.join(PKG, "libsop_hip.so"), f"-Wl,-rpath,{PKG}", "-Wl,--allow-shlib-undefined"])
    return exe


def _run(program, *args):
    r = subprocess.run([program, *args], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and "procedure ok" in r.stdout, (r.returncode, r.stdout[-2000:], r.stderr[-2000:])


@pytest.mark.parametrize("step", [("hipHostMalloc", 0), ("hipHostMalloc", 1), ("hipHostGetDevicePointer", 0), ("hipEventCreateWithFlags", 0)])
def test_a_failed_setup_is_made_up_for_by_the_next_call(program, step):
    _run(program, "setup", step[0], str(step[1]))


@pytest.mark.parametrize("call_fails", [0, 1])
def test_work_that_no_event_stands_behind_is_waited_for(program, call_fails):
    _run(program, "record", str(call_fails))


@pytest.mark.parametrize("first", [0, 1])
@pytest.mark.parametrize("shift", [0, 100])                      # (100: out of range, found by the first search)
def test_a_captured_call_is_refused_and_leaves_nothing(program, shift, first):
    _run(program, "captured", str(shift), str(first))
