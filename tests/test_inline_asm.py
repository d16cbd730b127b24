"""Inline assembly in the kernels, without a GPU.  The results of dot and matrix instructions want wait states
before some of their readers; the compiler keeps them only for instructions that it sees, so none of these
may stand in an asm statement."""
import glob
import os
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1803_03383_amd", "csrc")
SOURCES = sorted(glob.glob(os.path.join(CSRC, "*.hip")) + glob.glob(os.path.join(CSRC, "*.hpp")))


def _asm_texts(text):
    text = re.sub(r"//[^\n]*|/\*.*?\*/", "", text, flags=re.S)
    return re.findall(r"\basm\b(?:\s+volatile)?\s*\(\s*((?:\"(?:[^\"\\]|\\.)*\"\s*)+)", text)


@pytest.mark.parametrize("path", SOURCES, ids=os.path.basename)
def test_no_dot_or_matrix_instruction_in_inline_assembly(path):
    for asm in _asm_texts(open(path).read()):
        assert not re.search(r"\bv_(dot|mfma|smfmac)", asm), asm


def test_the_statements_are_found():
    found = [t for p in SOURCES for t in _asm_texts(open(p).read())]
    assert any("s_barrier" in t for t in found) and any("v_mad_i32_i24" in t for t in found)
