"""The host checks of large inputs where threads cannot be made (CPU only)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_checks_without_threads_or_memory_for_them(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("no host compiler")
    exe = str(tmp_path / "no_threads")
    subprocess.run(["g++", "-std=c++17", "-O2", "-I" + os.path.join(ROOT, "include"),
                    os.path.join(ROOT, "paper_2609_07204_amd", "csrc", "mc_host.cpp"),
                    os.path.join(ROOT, "tests", "sanitize", "no_threads.cpp"), "-o", exe, "-pthread"], check=True)
    p = subprocess.run([exe], stdout=subprocess.PIPE, stderr=subprocess.PIPE, text=True, timeout=60)
    assert p.returncode == 0 and p.stdout.split() == "kind 0 ok kind 1 ok".split(), (p.returncode, p.stdout, p.stderr)
