"""When the library counts as out of date, and what the launch tables may hold."""
import os
import re

import pytest

from paper_2505_22179_amd import build, tune


def test_every_kind_of_source_makes_the_library_stale(tmp_path, monkeypatch):
    csrc, include, lib = tmp_path / "csrc", tmp_path / "include", tmp_path / "lib.so"
    csrc.mkdir()
    include.mkdir()
    files = [csrc / "a.hip", csrc / "a.h", csrc / "plans.inc", include / "api.h"]
    for f in files + [lib]:
        f.write_text("")
    monkeypatch.setattr(build, "CSRC", str(csrc))
    monkeypatch.setattr(build, "INCLUDE", str(include))
    monkeypatch.setattr(build, "LIB", str(lib))
    for f in files:
        os.utime(f, (1000, 1000))
    os.utime(lib, (2000, 2000))
    assert not build.stale()
    for f in files:
        os.utime(f, (3000, 3000))
        assert build.stale(), f.name
        os.utime(f, (1000, 1000))
    lib.unlink()
    assert build.stale()


@pytest.mark.parametrize("table", ["tuned_plans.inc", "tuned_flat.inc"])
def test_every_row_of_a_table_is_among_the_tuners_candidates(table):
    """a row that the tuner does not try would be lost when it writes the table anew"""
    rows = re.findall(r"^\{([^}]*)\},", open(os.path.join(build.CSRC, table)).read(), flags=re.M)
    assert rows
    for row in rows:
        v = [int(t) for t in row.split(",")]
        if table == "tuned_flat.inc":
            N, K, _, tw, nw, ng, S, fused = v
            assert (tw, nw, 0, S, fused, 0, ng) in set(tune.flat_candidates(N, K)), row
            continue
        N, K, bucket = v[:3]
        for M in {0: (1, 4, 8), 1: (12, 16)}.get(bucket, (16 * bucket,)):   # the row counts the tuner times per bucket
            assert tuple(v[3:]) + (0,) in set(tune.candidates(N, K, M)), (row, M)
