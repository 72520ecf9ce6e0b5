"""The one-workgroup tails order their LDS accesses in both forms (CPU only; reads the sources).

A half-sweep of a tail level reads the 18 neighbours of a thread's cells and then overwrites the cells of its
colour, among them diagonal neighbours of other threads' cells. Reads and writes are kept apart by tail_sync:
a block barrier, or, where one wavefront owns the level, a wavefront fence. A form without it would
rest on the lanes' lockstep and on the compiler's order of one thread's accesses, and no run would show that
reliably, so the check is on the text: between the reads and the first write, and after the writes, every sweep
loop calls tail_sync<WAVE>() as a statement of its own, under no condition.
"""
import os
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1709_06350_amd", "csrc")
SYNC = re.compile(r"^\s*tail_sync<WAVE>\(\);", re.M)


@pytest.mark.parametrize("name", ["block_cycle.hip", "lin_block.h", "adj_block.hip"])
def test_sweeps_separate_reads_from_writes(name):
    text = re.sub(r"//[^\n]*", "", open(os.path.join(CSRC, name), encoding="utf-8").read())
    bodies = re.findall(r"void sweeps\(.*?\n  }\n", text, re.S)
    assert len(bodies) == 1, "one sweep loop a file"
    reads, writes = bodies[0].split("put(", 1)
    assert re.search(r"\b(source|off)\(", reads)
    assert SYNC.search(reads), "no unconditional tail_sync between the reads and the writes"
    assert SYNC.search(writes), "no unconditional tail_sync after the writes"
