"""Rules that the device sources keep and no run can show: a wait that a barrier
needs stands in one statement with it, where nothing can be moved between."""
from __future__ import annotations

import glob
import os
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2510_13847_amd", "csrc")
SOURCES = sorted(p for e in ("*.hip", "*.h", "*.cpp") for p in glob.glob(os.path.join(CSRC, e)))


@pytest.mark.parametrize("path", SOURCES, ids=os.path.basename)
def test_a_barrier_in_asm_waits_itself(path):
    text = re.sub(r"//[^\n]*", "", open(path).read())
    for m in re.finditer(r"__?asm(?:__)?\b[^;]*;", text):
        if "s_barrier" in m.group():
            assert re.search(r"s_waitcnt[^\"]*lgkmcnt\(0\).*s_barrier", m.group()), m.group()


def test_lanes_that_share_lds_words_are_ordered():
    """The row-streaming kernel writes a tile's pieces and reads other lanes'
    back without a barrier: an order of its own on both sides."""
    text = open(os.path.join(CSRC, "stream.hip")).read()
    write, read = text.index("if (writes) *reinterpret_cast<u32x4*>(wr"), text.index("*reinterpret_cast<const u32x4*>(rd")
    assert "wave_lds_order();" in text[write:read] and "wave_lds_order();" in text[:write]
