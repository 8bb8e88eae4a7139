"""The dense channel's host runtime and its memory pool on the CPU, compiled
from the library's own sources against stand-ins for HIP and the kernels."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "..", "paper_2608_07152_amd", "csrc")
ROCM = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "include")

pytestmark = pytest.mark.skipif(shutil.which("g++") is None or not os.path.isdir(os.path.join(ROCM, "hip")),
                                reason="needs g++ and the HIP headers")


def _run(tmp_path, test, sources):
    exe = tmp_path / "prog"
    subprocess.run(["g++", "-O1", "-g", "-std=c++17", "-pthread", "-D__HIP_PLATFORM_AMD__", "-Wno-attributes", "-w",
                    "-I", ROCM, "-I", CSRC, "-I", os.path.join(HERE, "..", "include"),
                    os.path.join(HERE, "native", test), *(os.path.join(CSRC, s) for s in sources), "-o", str(exe)],
                   check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.startswith("ok"), r.stdout + r.stderr


def test_a_failing_call_releases_no_busy_memory(tmp_path):
    _run(tmp_path, "handle_errors.cpp", ["pvs_api.cpp", "errors.cpp"])


def test_rules_of_the_memory_pool(tmp_path):
    _run(tmp_path, "dev_pool_rules.cpp", ["dev_pool.cpp"])


def test_memory_that_a_long_lived_index_holds(tmp_path):
    _run(tmp_path, "handle_memory.cpp", ["pvs_api.cpp", "dev_pool.cpp", "errors.cpp"])


def test_sparse_channel_beside_kept_memory(tmp_path):
    _run(tmp_path, "sparse_memory.cpp", ["pbm.cpp", "dev_pool.cpp", "errors.cpp"])


def test_how_far_ahead_scans_certify(tmp_path):
    _run(tmp_path, "reading_on.cpp", ["pvs_api.cpp", "dev_pool.cpp", "errors.cpp"])


def test_rows_of_the_threshold_sample(tmp_path):
    _run(tmp_path, "sample_rows.cpp", [])
