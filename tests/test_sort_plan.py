"""The sort's digit table fits the space that it is given (plain integer
arithmetic, CPU): every list of up to 6000 lines in plans of every size around
them, one to three passes of 8 to 10 bits, one and two intensity slots; and
larger plans around the powers of two."""
import ctypes
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
SRC = r"""
#include "sort_plan.h"
using namespace xs;
// entries and scan sums against the room of the place chosen, by the buffers'
// bytes: 1 fits, 0 not
static int fits(int64_t n, int64_t max_key, int64_t L, int64_t slots) {
  const SortPlan p = sort_plan(n, max_key, L, slots);
  const int64_t keys = p.few ? 1024 : 4096;
  if (p.entries != ((n + keys - 1) / keys) << p.rb) return 0;
  if (p.passes * p.rb < 63 && (max_key >> (p.passes * p.rb)) != 0) return 0;
  if (p.rb < 8 || p.rb > 10 || !p.col != (p.nblk > 64)) return 0;
  const int64_t table = 4 * p.entries, sums = p.col ? 0 : 4 * (p.entries / 1024 + 2);
  const int64_t hist = 4 * 256 * ((L + 4095) / 4096);
  switch (p.place) {
    case 0: return table <= hist && sums <= 4 * (hist / 4 / 1024 + 2);
    case 1: return table + sums <= 8 * L;
    case 2: return table + sums <= 8 * slots * 2 * 256;
  }
  return 0;
}
extern "C" int one(long long n, long long max_key, long long L, long long slots) { return fits(n, max_key, L, slots); }
extern "C" long long sweep(long long lo, long long hi, long long span, long long max_key, long long slots) {
  for (int64_t L = lo; L <= hi; ++L)
    for (int64_t n = L > span ? L - span : 0; n <= L; ++n)
      if (!fits(n, max_key, L, slots)) return L;
  return 0;
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("sort_plan")
    src, so = d / "s.cpp", d / "s.so"
    src.write_text(SRC)
    inc = os.path.join(os.path.dirname(HERE), "paper_2609_17273_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-O2", "-shared", "-fPIC", "-I", inc, str(src), "-o", str(so)], check=True)
    L = ctypes.CDLL(str(so))
    L.one.argtypes = [ctypes.c_longlong] * 4
    L.sweep.argtypes = [ctypes.c_longlong] * 5
    L.sweep.restype = ctypes.c_longlong
    return L


KEYS = [1, 200, 511, 512, 800, 1023, 1024, 3000, 1 << 17, (1 << 18) + 1, (1 << 20) - 1, 1 << 20, (1 << 30) - 1, (1 << 31) - 1]


@pytest.mark.parametrize("slots", [1, 2])
@pytest.mark.parametrize("max_key", KEYS)
def test_table_fits(lib, max_key, slots):
    assert lib.sweep(1, 6000, 1100, max_key, slots) == 0
    for b in range(13, 31):
        for L in (1 << b, (1 << b) + 1, (1 << b) - 1):
            for n in (L, L - 1, L // 2, 1025, 1, 0, min(L, 1 << 20), min(L, (1 << 20) + 1)):
                assert lib.one(n, max_key, L, slots), (n, L)


def test_two_blocks_of_ten_bits(lib):
    assert lib.one(1025, 800, 1025, 1)
