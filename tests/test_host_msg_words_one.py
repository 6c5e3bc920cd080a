"""The word-at-a-time form of the SHAKE256 blocks of mu = H(prefix || M), which the hash kernels with one
state per 16-lane row use, on the host under AddressSanitizer and UndefinedBehaviorSanitizer
(tests/msg_word_one.cpp): all misalignments, all lengths up to five blocks, the three prefixes."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_words_match_definition(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path / "msg_word_one")
    res = subprocess.run([gxx, "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined",
                          "-fno-sanitize-recover=all", "-I", os.path.join(ROOT, "paper_2211_12265_amd", "csrc"),
                          "-o", exe, os.path.join(ROOT, "tests", "msg_word_one.cpp")], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr
    res = subprocess.run([exe, "700"], capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, res.stdout + res.stderr
    assert res.stdout.count("cases=2804") == 3
