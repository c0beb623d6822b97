"""Accumulators where memory is short, on the CPU with a fake allocator.

A call of few cells keeps four copies of its next residues.  Where two buffers
of four do not fit it runs with one copy, and it must then hold no more than
that: a call that fits with one copy in each buffer is not refused because the
first buffer took room for four."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
OK, ENOMEM = 0, 2


@pytest.fixture(scope="module")
def fake(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("scratch") / "fake")
    subprocess.run(["g++", "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    os.path.join(ROOT, "tests", "scratch_fake.cpp"),
                    os.path.join(ROOT, "paper_2106_03058_amd", "csrc", "common.cpp"), "-o", exe], check=True)
    return exe


@pytest.mark.parametrize("budget,before,rc,copies,held", [
    (8000, 0, OK, 4, 8000),     # both buffers of four
    (7999, 0, OK, 1, 2000),     # the second does not fit
    (4500, 0, OK, 1, 2000),     # nor would one copy beside a first of four
    (3999, 0, OK, 1, 2000),     # nor the first
    (2000, 0, OK, 1, 2000),
    (4500, 1000, OK, 1, 2000),  # buffers of an earlier call with one copy
    (8000, 1000, OK, 4, 8000),
    (9000, 4500, OK, 4, 9000),  # larger ones of an earlier call
    (1999, 0, ENOMEM, 1, 1000),
])
def test_copies_fall_back_to_one(fake, budget, before, rc, copies, held):
    r = subprocess.run([fake, str(budget), "1000", str(before)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, (r.returncode, r.stdout, r.stderr)
    assert [int(v) for v in r.stdout.split()] == [rc, copies, held]
