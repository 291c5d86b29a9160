"""Host logic of calls that sum their pulses on a grid, without a GPU: scratch
sizes, sign-bit rows and plans of tests/host/drive_fold.cpp on the stand-in
runtime, with the host compiler's AddressSanitizer and
UndefinedBehaviorSanitizer."""

import os
import shutil
import subprocess

import pytest

from tests.test_host_abi import CXX, ROOT


@pytest.mark.skipif(shutil.which("ld") is None or not os.path.exists(CXX),
                    reason="no host linker or clang++")
def test_grid_scratch_and_sign_bit_rows(tmp_path):
    exe = tmp_path / "drive"
    res = subprocess.run(
        [CXX, "-std=c++17", "-g", "-O1", "-fno-omit-frame-pointer",
         "-fsanitize=address,undefined", "-fno-sanitize-recover=undefined",
         "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", f"-I{ROOT}/include",
         f"-I{ROOT}/paper_2311_18737_amd/csrc", "-o", str(exe),
         f"{ROOT}/tests/host/drive_fold.cpp",
         f"{ROOT}/paper_2311_18737_amd/csrc/ispl_api.cpp",
         f"{ROOT}/paper_2311_18737_amd/csrc/ispl_stream.cpp"], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-4000:]
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=0:allocator_may_return_null=1")
    run = subprocess.run([str(exe)], capture_output=True, text=True, env=env, timeout=300)
    assert run.returncode == 0, (run.stdout + run.stderr)[-4000:]
    assert "checks failed: 0, runtime errors: 0" in run.stdout
