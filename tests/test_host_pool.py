"""The pool of pinned host buffers, without a GPU: bounded, shared by all objects, given
back with the last one, and safe with several threads (ThreadSanitizer where it is there)."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2510_18221_amd", "csrc")


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
@pytest.mark.parametrize("checked", [False, True], ids=["plain", "tsan"])
def test_host_pool(tmp_path, checked):
    exe = str(tmp_path / "check")
    cmd = ["g++", "-std=c++17", "-O1", "-g", "-pthread", "-I" + CSRC, os.path.join(HERE, "host_pool_check.cpp"), "-o", exe]
    if checked:
        tsan = subprocess.run(["g++", "-print-file-name=libtsan.so"], capture_output=True, text=True).stdout.strip()
        if not os.path.isabs(tsan):
            pytest.skip("g++'s ThreadSanitizer runtime is not installed")
        cmd.insert(1, "-fsanitize=thread")
    subprocess.run(cmd, check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=100)
    if checked and "unexpected memory mapping" in r.stderr:
        pytest.skip("ThreadSanitizer cannot map its memory on this kernel")
    assert r.returncode == 0, r.stdout + r.stderr
