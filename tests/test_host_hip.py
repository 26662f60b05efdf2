"""The library's host code on the CPU, over a stand-in HIP runtime
(tests/native/fake_hip.cpp): what it calls under capture, what it keeps and
frees, and what it does when calls fail.  Each case of fake_hip_cases.py runs
in a process of its own."""

import os
import shutil
import subprocess
import sys

import pytest

from paper_2401_14351_amd import binding

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")

pytestmark = [pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available"),
              pytest.mark.skipif(not os.path.exists(binding.LIB_PATH), reason="libsllm.so not built")]


@pytest.fixture(scope="module")
def fake(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("fake") / "libfakehip.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-shared", "-fPIC", f"-I{ROCM}/include",
                    f"-I{os.path.join(ROOT, 'include')}", f"-I{os.path.join(os.path.dirname(binding.LIB_PATH), 'csrc')}",
                    os.path.join(HERE, "native", "fake_hip.cpp"), "-o", so], check=True)
    return so


def run(fake, tmp_path, case):
    r = subprocess.run([sys.executable, os.path.join(HERE, "fake_hip_cases.py"), fake, case, str(tmp_path)],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.strip().endswith("ok"), r.stdout + r.stderr


@pytest.mark.parametrize("case", ["events_under_capture", "close_after_capture", "open_under_capture", "refused_free", "failure_under_capture",
                                  "error_not_left_pending", "idle_blocks", "tables_are_checked",
                                  "staging_sizes", "scatter_unroll", "pack_sizes", "plan_writers"])
def test_host_code(fake, tmp_path, case):
    run(fake, tmp_path, case)
