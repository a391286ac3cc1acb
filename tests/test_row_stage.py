"""The words of a row that the rows' pass brings into LDS (csrc/row_stage.h,
compiled here for the host): all of a row's words or none, and never one past a
pool that ended before the rows did (the rows that did not fit have count 0 and
the offsets they would have had)."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

import oracle
from paper_2602_19873_amd import workloads

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2602_19873_amd", "csrc")


@pytest.fixture(scope="module")
def stage(tmp_path_factory):
    d = tmp_path_factory.mktemp("row_stage")
    src = d / "s.cc"
    src.write_text('#include "row_stage.h"\nextern "C" unsigned stage(unsigned off, unsigned cnt, unsigned next) '
                   '{ return sfcnl::row_stage_words(off, cnt, next); }\n')
    so = d / "s.so"
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, "-o", str(so), str(src)], check=True)
    f = C.CDLL(str(so)).stage
    f.argtypes, f.restype = [C.c_uint] * 3, C.c_uint
    return f


@pytest.mark.parametrize("n,target,cut_row", [(500, 20.0, 243), (500, 20.0, 0), (500, 20.0, 499), (700, 300.0, 350),
                                              (700, 600.0, 10)])
def test_short_pool(stage, n, target, cut_row):
    s = workloads.uniform_varied(n, 3, target=target)
    perm = oracle.sfc_order(oracle.hilbert_keys(s.x, s.y, s.z, s.box)).astype(np.int64)
    info, pool = oracle.row_list(*(np.ascontiguousarray(a[perm]) for a in (s.x, s.y, s.z, s.h)), True)
    info = info.astype(np.int64)
    ends = np.append(info[1:, 0], len(pool))
    words = int(info[cut_row, 0]) + 1  # the pool ends inside row cut_row
    cnt = np.where(ends <= words, info[:, 1], 0)
    for i in range(n - 1):
        got = stage(int(info[i, 0]), int(cnt[i]), int(info[i + 1, 0]))
        assert got in (0, ends[i] - info[i, 0])
        assert got == 0 or info[i, 0] + got <= words, "row %d of {%d, %d} reads %d words" % (i, info[i, 0], cnt[i], got)
        assert cnt[i] == 0 or got or ends[i] - info[i, 0] > 256


@pytest.mark.parametrize("off,cnt,nxt,want", [
    (10, 5, 13, 3), (10, 5, 10, 0), (10, 5, 11, 0), (10, 64, 12, 2), (10, 65, 13, 0), (10, 65, 14, 4), (10, 0, 14, 0),
    (10, 300, 266, 256), (10, 300, 267, 0), (300, 5, 10, 0), (0xFFFFFFF0, 3, 0xFFFFFFF4, 4)])
def test_edges(stage, off, cnt, nxt, want):
    assert stage(off, cnt, nxt) == want
