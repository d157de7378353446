"""The layout of a weight-gradient launch (csrc/tn_plan.h, plain C++): every chunk of every problem is worked on by one XCD, the
queues are as the kernel reads them, and no chunk is longer than the plan says.  No GPU is touched."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2307_07649_amd", "csrc")
SOURCE = r"""
#include "tn_plan.h"
using namespace tgnn;
// shape: n rows {rows, counted, n, k, heads, tiles}.  mine [8, n], begin [8, 16], order [16], word [n] -> the longest queue
extern "C" int plan(const int* shape, int n, unsigned long long* mine, int* begin, int* order, int* word) {
  TnShape p[TN_MAX_GROUP];
  for (int i = 0; i < n; ++i, shape += 6) p[i] = TnShape{shape[0], shape[1] != 0, shape[2], shape[3], shape[4], shape[5]};
  TnPlan q;
  const int longest = tn_place(q, p, n, tn_chunk_units(p, n) * TN_ROWS);
  for (int x = 0; x < 8; ++x) {
    for (int i = 0; i < n; ++i) mine[x * n + i] = q.mine[x][i];
    for (int t = 0; t < 16; ++t) begin[x * 16 + t] = q.qbegin[x][t];
  }
  for (int t = 0; t < 16; ++t) order[t] = q.qprob[t];
  for (int i = 0; i < n; ++i) word[i] = q.chunks[i];
  return longest;
}
extern "C" int chunk_rows(int rows, int chunks) { return tn_chunk_rows(rows, chunks); }
extern "C" int max_rows() { return TN_MAX_ROWS; }
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    (d / "plan.cpp").write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC, str(d / "plan.cpp"), "-o", str(d / "plan.so")],
                   check=True)
    return ctypes.CDLL(str(d / "plan.so"))


def pieces(n):
    return (n + 63) // 64


def problem(rows, n, k, counted=False, heads=1):
    return [rows, int(counted), n, k, heads, heads * pieces(n) * pieces(k)]


def check(lib, shapes):
    """Walks the queues as the kernel does; returns the longest one and the rows of a chunk per problem."""
    n = len(shapes)
    s = np.array(shapes, np.int32)
    mine, begin = np.zeros((8, n), np.uint64), np.zeros((8, 16), np.int32)
    order, word = np.zeros(16, np.int32), np.zeros(n, np.int32)
    ptr = lambda a: a.ctypes.data_as(ctypes.c_void_p)
    longest = lib.plan(ptr(s), n, ptr(mine), ptr(begin), ptr(order), ptr(word))
    chunks, shift = word & 0xffffff, word >> 24
    done = [set() for _ in range(n)]
    for x in range(8):
        assert sorted(order[:n]) == list(range(n)) and begin[x, 0] == 0 and np.all(begin[x, n + 1:] == 0x7fffffff)
        for o in range(n):
            i = order[o]
            bits = [b for b in range(64) if int(mine[x, i]) >> b & 1]
            for local in range(begin[x, o + 1] - begin[x, o]):
                nth, tile = divmod(local, s[i, 5])
                chunk = (bits[nth >> shift[i]] << shift[i]) + (nth & ((1 << shift[i]) - 1))
                assert chunk < chunks[i] and (chunk, tile) not in done[i]
                done[i].add((chunk, tile))
    rows = []
    for i in range(n):
        assert len(done[i]) == chunks[i] * s[i, 5]
        rows.append(lib.chunk_rows(int(s[i, 0]), int(chunks[i])))
        assert rows[-1] * chunks[i] >= s[i, 0]
    assert longest == begin[:, n].max()
    return longest, rows


# shapes of a training step, of a stand-alone backward call, of narrow widths
@pytest.mark.parametrize("rows,est", [(1, 1), (96, 64), (600, 825), (1800, 2475), (12000, 16500), (4800, 19800)])
@pytest.mark.parametrize("dm,dt,de,H", [(100, 100, 172, 2), (32, 32, 16, 1), (200, 100, 172, 4), (4, 1, 0, 2)])
def test_step(lib, rows, est, dm, dt, de, H):
    C = de + dt
    d_in = 2 * dm + dt + de
    shapes = [problem(rows, 2 * dm, dm + 1), problem(rows, dm, dm), problem(rows, dm // H + 3, C, heads=H), problem(rows, dm // H + 3, C, heads=H),
              problem(rows, 2 * dt, 1), problem(est, 2 * dm, dm + 1, True), problem(est, 2 * dm, dm + 1, True),
              problem(est, 3 * dm, d_in + 1, True), problem(est, 3 * dm, dm + 1, True)]
    longest, _ = check(lib, shapes)
    assert longest >= 1


# more rows than 64 chunks hold: as many chunks as it takes, none longer than the longest that the plan looks at
@pytest.mark.parametrize("rows", [131072, 131073, 132000, 262145, 480000, 1000001])
def test_long_problems(lib, rows):
    for dm, k in ((4, 4), (8, 11), (100, 100)):
        shapes = [problem(rows // 11, dm, dm), problem(rows, 2 * dm, dm + 1), problem(rows, 2 * dm, k + 1)]
        _, per_chunk = check(lib, shapes)
        assert max(per_chunk) <= lib.max_rows(), per_chunk


# no more than 64 chunks add to a tile as long as their length does not exceed 2,048 rows (narrow problems, whose queues would
# take more)
@pytest.mark.parametrize("rows", [8192, 8193, 19404, 60000, 131071, 131072, 131073, 200000])
@pytest.mark.parametrize("dm,dt,de,H", [(34, 53, 71, 2), (4, 1, 0, 2), (16, 16, 8, 1)])
def test_chunks_of_a_tile(lib, rows, dm, dt, de, H):
    R = rows // 11
    shapes = [problem(R, dm, dm), problem(R, dm // H + 3, de + dt, heads=H), problem(R, 2 * dt, 1), problem(rows, 2 * dm, dm + 1),
              problem(rows, 2 * dm, dm + 1)]
    _, per_chunk = check(lib, shapes)
    for s, rows_per in zip(shapes, per_chunk):
        assert -(-s[0] // rows_per) <= max(64, -(-s[0] // 2048)), (s, rows_per)
