"""Loops that go over edges, slots or vertices in steps of a whole grid count in
64 bits: a graph may hold up to 2^32 - 1 edges, and a 32-bit counter that steps
past the end wraps around and never ends."""
import glob
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2010_08423_amd", "csrc")
# Counters that cannot come near 2^32: runs of a scan (at most 16384), and the
# evaluation form's lists, whose prefix state takes over 1 KB per edge.
BOUNDED = {("rs_coef.hip", "run"), ("rs_compact.hip", "j")}
LOOP = re.compile(r"for \(uint32_t (\w+) = [^;]*blockIdx[^;]*;[^;]*; \1 \+= gridDim")


def test_grid_steps_do_not_wrap():
    found = {(os.path.basename(f), m.group(1)) for f in glob.glob(os.path.join(CSRC, "*.h*")) for m in LOOP.finditer(open(f).read())}
    assert found <= BOUNDED
