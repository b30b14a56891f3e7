"""The host side of the C-ABI without a GPU: ``tests/native/api_check.cpp`` runs lbrb_api.cpp on a HIP
runtime of its own (host memory, launches counted, timed by a fixed clock or failing), built with
AddressSanitizer and UndefinedBehaviorSanitizer (host code only)."""
import os
import shutil
import subprocess

import pytest

from tests.test_sanitizers import ROOT, SAN

pytestmark = pytest.mark.skipif(shutil.which("g++") is None or not os.path.isdir("/opt/rocm/include"),
                                reason="needs g++ and the HIP headers")


@pytest.fixture(scope="module")
def api_check(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("api") / "api_check")
    csrc = os.path.join(ROOT, "paper_1604_01829_amd", "csrc")
    cmd = (["g++", "-std=c++17", "-Wall", "-Wextra", "-Wno-unknown-pragmas", "-D__HIP_PLATFORM_AMD__",
            "-I/opt/rocm/include"] + SAN +
           [os.path.join(ROOT, "tests", "native", "api_check.cpp"), os.path.join(csrc, "lbrb_api.cpp"),
            os.path.join(csrc, "lbrb_plan.cpp"), "-o", exe])
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    return exe


def _run(exe, what):
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=1:abort_on_error=0:halt_on_error=1",
               UBSAN_OPTIONS="print_stacktrace=1:halt_on_error=1")
    r = subprocess.run([exe, what], capture_output=True, text=True, timeout=300, env=env)
    assert r.returncode == 0, (r.stdout + r.stderr)[-4000:]
    assert f"{what} ok" in r.stdout


def test_autotuner_times_the_moving_wall_links(api_check):
    _run(api_check, "tune")


def test_a_failing_launch_of_a_replay_is_reported(api_check):
    _run(api_check, "replay")


def test_observables_allocate_nothing(api_check):
    _run(api_check, "observe")
