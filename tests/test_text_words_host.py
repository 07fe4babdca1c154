"""The recognizers' word arithmetic (paper_2606_15650_amd/csrc/text_words.hpp)
on the CPU, up to the largest text that recognize_spans accepts, built with
g++ under the address and undefined-behaviour sanitizers."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_words_up_to_the_largest_text(tmp_path):
    exe = str(tmp_path / "text_words")
    b = subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
                        "-I" + os.path.join(ROOT, "paper_2606_15650_amd", "csrc"),
                        os.path.join(ROOT, "tests", "native", "text_words_test.cpp"), "-o", exe],
                       capture_output=True, text=True)
    assert b.returncode == 0, b.stderr
    env = {k: v for k, v in os.environ.items() if k != "LD_PRELOAD"}
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120, env=env)
    assert r.returncode == 0, r.stdout + r.stderr
    assert "ALL PASSED" in r.stdout
