"""Every shipped tuner choice is one the library can look up.

The tuners keep the records of meshes whose n / 2 is a multiple of 48 or 40 apart (kind .v2, made with the tiles
of 48 and 40 columns among the candidates) from those of the other meshes (.v1). A shipped row under the
other version is never read: the first use on a fresh machine then times its candidates, and two machines
may choose differently. The batched workload's meshes (boxes of 64^3, 96^3 and 128^3 and their coarse levels)
are all shipped, and on the GPU the shipped choice of 96^3 is used untimed.
"""
import os
import struct

import pytest

from paper_1709_06350_amd import mr

PATH = os.path.join(os.path.dirname(mr.__file__), "tuning_defaults.txt")


def _rows():
    return [ln.strip().split("|") for ln in open(PATH) if ln.strip() and not ln.startswith("#")]


def test_every_row_is_under_the_kind_that_its_size_is_looked_up_by():
    for kind, _, _, _, n, _ in _rows():
        wide = (int(n) // 2) % 48 == 0 or (int(n) // 2) % 40 == 0
        assert kind.endswith(".v2" if wide else ".v1"), (kind, n)


def test_the_batched_workloads_meshes_are_shipped():
    shipped = {int(r[4]) for r in _rows() if r[0].startswith("blin32.")}
    assert {128, 64, 32, 16, 8, 96, 48, 24, 12} <= shipped
    assert any(r[0] == "blin32.v2" and r[4] == "96" for r in _rows())


@pytest.mark.gpu
def test_shipped_choice_of_96_is_used_untimed(tmp_path):
    from gpu_util import announce, require_gpu
    require_gpu()
    announce("shipped tuner choice, 96^3")
    row = next(r for r in _rows() if r[0] == "blin32.v2" and r[4] == "96")
    vals = [int(v) for v in row[5].split(",")]
    mr.tuning_file(str(tmp_path / "fresh.txt"))
    try:
        tm, tj, ci, ms = mr.tune_lin_tiles(96)
    finally:
        mr.tuning_file(None)
    assert [tm, tj, ci] == vals[:3]
    assert struct.unpack("i", struct.pack("f", ms))[0] == vals[7]   # the recorded time, not a new one
