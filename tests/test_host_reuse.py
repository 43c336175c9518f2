"""When calls run directly, capture a graph or replay it (csrc/reuse.h)."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def reuse(tmp_path_factory):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path_factory.mktemp("reuse") / "reuse_check")
    subprocess.run([cxx, "-std=c++17", "-O1", "-Wall", "-Werror", os.path.join(HERE, "host", "reuse_check.cpp"), "-o",
                    exe], check=True)
    return lambda keys: subprocess.run([exe], input=keys + "\n", capture_output=True, text=True, check=True).stdout


@pytest.mark.parametrize("keys,acts", [
    ("AAAAAA", "dddcrr"),
    ("AAAABBBBAAAAA", "dddcdddcdddcr"),
    ("ABABABABAB", "dddddddddd"),
    # inputs that alternate leave the captured graph alone
    ("AAAABABABABABABAB", "dddcdrdrdrdrdrdrd"),
    ("AAAABBBABBBAB", "dddcdddrdddrd"),
    ("AAABAAAA", "ddddddd" + "c"),
])
def test_capture_rule(reuse, keys, acts):
    assert reuse(keys) == acts
