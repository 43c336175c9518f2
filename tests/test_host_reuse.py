"""When calls run directly, capture a graph or replay it, and when registrations
do without the one-launch loop (csrc/reuse.h)."""
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
    return lambda *a: subprocess.run([exe, *a], capture_output=True, text=True, check=True).stdout


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
    assert reuse("capture", keys) == acts


def test_loop_rule(reuse):
    """One stall, 255 calls without the loop, then the loop again."""
    assert reuse("loop", "....") == "llll"
    assert reuse("loop", "." + "s" * 258) == "ll" + "i" * 255 + "li"


@pytest.mark.parametrize("text,limit", [(None, 200000), ("1", 1), ("5000", 5000), ("", 200000), ("abc", 200000),
                                        ("0", 200000), ("-3", 200000), ("12x", 200000), ("1e6", 200000),
                                        ("99999999999", 200000), ("99999999999999999999", 200000), (" 7", 200000)])
def test_poll_limit(reuse, text, limit):
    assert int(reuse("limit", *([] if text is None else [text]))) == limit
