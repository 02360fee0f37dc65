"""The committed tuner cache and the measured traffic hold for the sources that they were taken with, all of them."""
import os
import shutil
import sys

import pytest

from paper_2609_05528_amd import build_lib

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCES = ("operator.hip", "adjoint_cells.hip", "rtt_internal.h", "tables.cpp")


def bench():
    sys.path.insert(0, ROOT)
    import bench
    return bench


@pytest.mark.parametrize("name", SOURCES)
def test_every_source_of_the_operator_counts(tmp_path, name):
    csrc = tmp_path / "csrc"
    shutil.copytree(build_lib.CSRC, csrc)
    assert build_lib.operator_digest(str(csrc)) == build_lib.operator_digest()
    with open(csrc / name, "a") as f:
        f.write("\n")
    assert build_lib.operator_digest(str(csrc)) != build_lib.operator_digest()
    assert build_lib.tune_cache_header(str(csrc)) != build_lib.tune_cache_header()


def test_bench_ignores_a_cache_made_with_other_sources(tmp_path, monkeypatch):
    b = bench()
    assert b.source_digest() == build_lib.operator_digest()
    own, other = build_lib.tune_cache_header(), build_lib.tune_cache_header().rsplit(" ", 1)[0] + " 0123456789abcdef\n"
    for head, used in ((other, False), (own.split(" sources")[0] + "\n", False), (own, True)):
        path = tmp_path / "cache.txt"
        path.write_text(head + "0 1 4 11\n")
        monkeypatch.setattr(b, "TUNE_CACHE", str(path))
        monkeypatch.setattr(b, "_tune_cache_copy", None)
        got = b.tune_cache()
        assert (got is not None) == used, head
        if got:
            os.remove(got)
    monkeypatch.setattr(b, "_tune_cache_copy", None)
