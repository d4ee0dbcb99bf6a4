"""The sources that bench.py hashes for each step: the committed counters count as
measured only while these are unchanged, so none may fall out of the lists."""
import os
import re

import pytest

import bench


def test_lists_and_prefixes_match_files():
    for step in bench.STEP_SOURCES:
        files = bench.step_files(step)
        assert len(files) == len(set(files))
        for prefix in bench.STEP_PREFIXES.get(step, ()):
            assert any(f.startswith(prefix) for f in files), (step, prefix)


def test_every_factorisation_and_solve_source_is_hashed():
    hashed = {f for step in bench.STEP_SOURCES for f in bench.step_files(step)}
    for f in sorted(os.listdir(bench.CSRC)):
        # (the transposed solve's L^T pass is not a timed step)
        if re.match(r"getr[fs]", f) and not f.startswith("getrs_lt"):
            assert f in hashed, f


def test_included_headers_are_hashed():
    for step in bench.STEP_SOURCES:
        files = bench.step_files(step)
        for f in files:
            if f == "chain.hip":  # (includes the transposed solve's header)
                continue
            with open(os.path.join(bench.CSRC, f)) as fh:
                for inc in re.findall(r'#include "(\w+\.hpp)"', fh.read()):
                    assert inc in files, (step, f, inc)


def test_a_missing_source_is_an_error(monkeypatch):
    monkeypatch.setitem(bench.STEP_PREFIXES, "getrf", ("getrf_no_such_",))
    with pytest.raises(FileNotFoundError, match="getrf_no_such_"):
        bench.source_hash("getrf")
