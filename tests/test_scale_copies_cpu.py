"""The copies of the MXFP4 tiles, run on the host lane by lane (host/scale_copies.cpp): the headers that the kernel includes, with the copies
themselves recorded instead of done."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HOST = os.path.join(ROOT, "tests", "host")
CSRC = os.path.join(ROOT, "paper_2601_07475_amd", "csrc")


@pytest.fixture(scope="module")
def counts(tmp_path_factory):
    """What the program counted over every tile, full and ragged, and 22 numbers of blocks a row."""
    if not shutil.which("g++"):
        pytest.skip("no host compiler")
    out = tmp_path_factory.mktemp("scale_copies")
    for name in ("scale_chunks.h", "code_rows.h"):      # by themselves, so that they find the host's lds_dma.h
        shutil.copy(os.path.join(CSRC, name), out)
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wno-unknown-pragmas", f"-I{out}", f"-I{HOST}", os.path.join(HOST, "scale_copies.cpp"), "-o", out / "run"],
                   check=True, timeout=300)
    text = subprocess.run([out / "run"], check=True, capture_output=True, text=True, timeout=300).stdout
    return {k: int(v) for k, v in re.findall(r"(\w+) (\d+)", text)}


def test_a_unit_finds_its_scale_bytes(counts):
    """Whether copies land at once or as late as the waits allow."""
    assert counts["checked"] > 5e7 and counts["wrong"] == 0


def test_copies_of_a_chunk_agree_where_they_overlap(counts):
    """Copies in flight land in no order that the program may rely on: two that write one place bring the same bytes."""
    assert counts["differ"] == 0


def test_scalar_offsets_stay_within_the_operand(counts):
    """A buffer's range check compares with its length less the scalar offset: rows past the edge of an operand, and chunks past the end of
    its last row, must not make that negative."""
    assert counts["past"] == 0
