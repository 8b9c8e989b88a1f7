"""The server's one device block on the host: its bytes are the sum of its
arrays as the header documents them (what the budget check and the reported
state bytes count), no two arrays overlap, and each starts aligned to its
elements."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = r"""
#include "serve_layout.h"
using namespace odp;
extern "C" int layout(uint64_t cap, uint64_t (*a)[3]) {  // offset, bytes, alignment of each array
  const ServerLayout L = server_layout(cap);
  int n = 0;
  auto put = [&](uint64_t at, uint64_t bytes, uint64_t align) { a[n][0] = at; a[n][1] = bytes; a[n++][2] = align; };
  for (int i = 0; i < 2; ++i) {
    put(L.stage[i], 1024 * (64 + 8 + 8 + 1), 256);  // (copied from the host)
    put(L.dig[i], 1024 * 8, 8);
    put(L.pend[i], cap * 32, 8);
  }
  put(L.log, cap * 64, 64);
  put(L.kstart, 11 * cap * 8, 8);
  put(L.kmaxend, 11 * cap * 8, 8);
  put(L.link, cap * 4, 4);
  put(L.kc_at, cap * 4, 4);
  uint64_t slots = 1024;
  while (slots < 2 * cap) slots *= 2;
  for (int i = 0; i < 6; ++i) put(L.tables[i], slots * 40, 8);
  put(L.st, sizeof(ServeState), 8);
  put(L.known, (cap + 8) & ~3ull, 4);
  put(L.zeroed, 0, 1);
  put(L.bytes, 0, 1);
  return n;
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("layout")
    (d / "layout.cpp").write_text(SOURCE)
    so = str(d / "layout.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_2601_12713_amd", "csrc"), "-o", so, str(d / "layout.cpp")], check=True)
    return ctypes.CDLL(so)


@pytest.mark.parametrize("cap", [1, 2, 3, 7, 255, 256, 257, 511, 512, 513, 1000, 4097, 65535, 10_000_000, 2**32 - 1])
def test_block_is_the_sum_of_its_arrays(lib, cap):
    out = ((ctypes.c_uint64 * 3) * 64)()
    n = lib.layout(ctypes.c_uint64(cap), out)
    rows = [tuple(out[i]) for i in range(n)]
    (zeroed, _, _), (total, _, _) = rows[-2:]
    arrays = sorted(rows[:-2])
    assert sum(b for _, b, _ in arrays) == total
    at = 0
    for off, nbytes, align in arrays:
        assert off == at and off % align == 0, (off, at, align)
        at += nbytes
    assert at == total
    # the tables, the state and the flags start at zero: everything from `zeroed` on
    assert [a for a in arrays if a[0] >= zeroed] == arrays[-8:]
