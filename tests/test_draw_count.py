"""The vector instructions of a draw that bench.py prices the level kernel by
are those of the draw as it is: counted in the assembly of draw-only loops."""
import os
import re
import shutil
import subprocess

import pytest

import bench
from paper_2106_03058_amd import build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    if shutil.which("hipcc") is None:
        pytest.skip("no hipcc")
    out = str(tmp_path_factory.mktemp("draws") / "draws.asm")
    subprocess.run(["hipcc", "-x", "hip", *build.FLAGS, "--cuda-device-only", "-S",
                    os.path.join(ROOT, "tests", "draw_loop.hip"), "-o", out], check=True, capture_output=True)
    with open(out) as f:
        return f.read()


@pytest.mark.parametrize("loop,count", [
    ("draws_a0", bench.VALU_PER_DRAW_A0),
    ("draws_ap", bench.VALU_PER_DRAW),
    ("draws_dense", bench.VALU_PER_DRAW + bench.VALU_DENSE_SKIP),
])
def test_vector_instructions_of_a_draw(assembly, loop, count):
    body = assembly[assembly.index(f"\n{loop}:"):]
    body = body[:body.index("s_endpgm")]
    body = body[body.index("Loop Header"):]
    body = body[:body.index("s_cbranch")]
    assert len(re.findall(r"^\s+v_\w+", body, re.M)) == count
