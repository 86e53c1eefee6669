"""Ordering of the library's host side (csrc/tnsim_abi.cpp) on a stream of its
own, against a stand-in for the HIP runtime whose streams are slow queues
(tests/fake_hip.cpp): what a call hands back has been computed by then, and
nothing is freed that work in flight still uses, nothing is launched whose
result is not read.  No GPU."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ABI = os.path.join(ROOT, "paper_2601_04422_amd", "csrc", "tnsim_abi.cpp")
ROCM = "/opt/rocm/include"

pytestmark = pytest.mark.skipif(shutil.which("g++") is None or not os.path.isdir(ROCM),
                                reason="needs g++ and the HIP headers")


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("fake_hip") / "fake_hip")
    # two names that only hipcc knows
    subprocess.check_call(
        ["g++", "-std=c++17", "-O1", "-w", "-pthread", "-D__HIP_PLATFORM_AMD__",
         "-D__align__(x)=__attribute__((aligned(x)))", "-DHIP_SYMBOL(x)=(&(x))", "-I", ROCM,
         "-I", os.path.join(ROOT, "include"), "-o", out,
         os.path.join(ROOT, "tests", "fake_hip.cpp"), ABI])
    return out


def _run(exe, scenario):
    r = subprocess.run([exe, scenario], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout + r.stderr


def test_gradient_is_read_after_its_adjoints(exe):
    _run(exe, "gradient")


def test_a_replaced_graph_stays_until_its_sweep_is_done(exe):
    _run(exe, "replan")


def test_no_factors_of_the_second_q(exe):
    _run(exe, "qr")
