"""The cut of ranges into sieve segments and the word indices, as the library's own host
code does them, on the CPU: every integer's index turns back into that integer."""
import os
import shutil
import subprocess

import pytest

from paper_2506_01099_amd import build as hip_build

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host C++ compiler")
def test_word_indices_turn_back_into_their_integers(tmp_path):
    exe = tmp_path / "segments"
    rocm = os.path.dirname(os.path.dirname(hip_build.hipcc()))
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I" + os.path.join(rocm, "include"),
                           "-I" + os.path.join(hip_build.HERE, "csrc"), "-o", str(exe),
                           os.path.join(HERE, "segments_driver.cpp")])
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    assert out.returncode == 0 and out.stdout.startswith("ok"), out.stdout + out.stderr
    assert int(out.stdout.split()[1]) > 10**6
