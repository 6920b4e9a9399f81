"""Host check of the copy of results to the caller's arrays (host_copy.cpp), compiled
with g++ against stand-ins for the HIP runtime (tests/cpp/copy_check.cpp): every byte
arrives, also where a chunk does not divide evenly among the threads that empty it."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2605_30355_amd", "csrc")


@pytest.fixture(scope="module")
def checker(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("bin") / "copy_check")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-pthread", "-I",
                           os.path.join(ROOT, "include"), "-I", CSRC, "-D__HIP_PLATFORM_AMD__",
                           "-I", "/opt/rocm/include",
                           os.path.join(ROOT, "tests", "cpp", "copy_check.cpp"),
                           os.path.join(CSRC, "host_copy.cpp"), "-o", out])
    return out


def lines(checker, lengths, device=0, busy_ms=0):
    r = subprocess.run([checker, str(device), str(busy_ms), *map(str, lengths)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr
    got = [dict(kv.split("=") for kv in line.split()) for line in r.stdout.splitlines()]
    assert [int(g["len"]) for g in got] == list(lengths)
    return got


def run(checker, lengths, device=0):
    return [int(g["len"]) for g in lines(checker, lengths, device) if g["bad"] != "0"]


def test_lengths_around_every_share(checker):
    """Last chunks of a few bytes, and of a few more or fewer than a multiple of 4096
    bytes per thread, for 2 to 8 threads, at either chunk size."""
    lengths = [0, 1, 196608, 196609, 2621440]
    for whole in (5 << 19, 9 << 19, 4 << 21, 5 << 21):  # full chunks before the last one
        for of in range(2, 9):
            for r in (1, of - 1, of, 4096 * of - 1, 4096 * of, 4096 * of + 1, 5 * 4096 * of + of - 1):
                lengths.append(whole + r)
    # 753 x 3601, 1003 x 3267 and 271 x 271 x 999 spins
    lengths += [753 * 3601, 1003 * 3267, 271 * 271 * 999]
    assert run(checker, lengths) == []


def test_stream_of_another_device(checker):
    """Results of a batch may be asked for with another device current than its own."""
    assert run(checker, [800, 200000, 3 << 20, 20 << 20], device=1) == []


def test_the_threads_sleep_while_the_device_works(checker):
    """Results are asked for while sweeps still run; a long trial must not cost its time on
    every copying thread."""
    for g in lines(checker, [3 << 20, 20 << 20], busy_ms=400):
        assert g["bad"] == "0" and float(g["cpu_ms"]) < 200.0, g
