"""The index arithmetic of the dense local pass (csrc/eik_walk.hpp), on the CPU
under the undefined-behaviour sanitizer: every plane once, none outside."""

import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_walks_cover_the_grid(tmp_path):
    exe = str(tmp_path / "walk_driver")
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-fsanitize=undefined", "-fno-sanitize-recover=all",
                    "-o", exe, os.path.join(HERE, "sanitize", "walk_driver.cpp")], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and "clean" in r.stdout, r.stdout + r.stderr
