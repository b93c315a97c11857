"""The conversion of spins between the caller's bytes and the packed bits, which runs on
several host threads from 2^21 sites: compared with one site at a time over many calls
(a thread that touched another's byte would lose bits now and then), and under the
thread sanitizer.  Octant edges of 4 modulo 8 end their rows, and the octant, in half
a byte."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SHAPES = [(128, 8), (144, 24), (160, 40), (128, 16), (160, 32), (168, 56)]


def _build(tmp, *flags):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("g++ not available")
    exe = str(tmp / "check")
    subprocess.run([cxx, "-O2", "-std=c++17", "-pthread", *flags, "-I", os.path.join(ROOT, "paper_1005_4713_amd", "csrc"),
                    "-o", exe, os.path.join(ROOT, "tests", "spin_bytes_check.cpp")], check=True, capture_output=True)
    return exe


@pytest.fixture(scope="module")
def plain(tmp_path_factory):
    return _build(tmp_path_factory.mktemp("plain"))


@pytest.fixture(scope="module")
def sanitized(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("tsan")
    try:
        exe = _build(tmp, "-g", "-fsanitize=thread")
    except subprocess.CalledProcessError:
        pytest.skip("no thread sanitizer")
    if subprocess.run([exe, "8", "8", "1"], capture_output=True).returncode:
        pytest.skip("the thread sanitizer does not run here")
    return exe


@pytest.mark.parametrize("L,d,calls", [(8, 8, 1), (24, 24, 1), (48, 16, 1), (128, 8, 1500)] +
                         [(L, d, 20) for L, d in SHAPES[1:]])
def test_packed_as_site_by_site(plain, L, d, calls):
    out = subprocess.run([plain, str(L), str(d), str(calls)], capture_output=True, text=True, check=True).stdout
    assert int(out) == 0


@pytest.mark.parametrize("L,d", SHAPES)
def test_no_data_race(sanitized, L, d):
    run = subprocess.run([sanitized, str(L), str(d), "2"], capture_output=True, text=True)
    assert run.returncode == 0, run.stderr[:2000]
    assert int(run.stdout) == 0
