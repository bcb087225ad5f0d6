"""Rules that the kernels and the launch code share, compiled for the host and compared with their
definitions over all forms they accept (no GPU)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def run_host(tmp_path, text):
    """Compiles a program against the kernel sources' plain headers and runs it; its output."""
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(text)
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Wno-unknown-pragmas", "-I",
                    os.path.join(ROOT, "paper_1409_6070_amd", "csrc"), str(src), "-o", str(exe)], check=True, timeout=120)
    return subprocess.run([str(exe)], check=True, timeout=120, stdout=subprocess.PIPE, text=True).stdout


BIT_ROWS = r"""
#include "bit_rows.h"
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>
using namespace sscn;
typedef std::vector<uint64_t> Row;
static bool bit(const Row& r, int i) { return r[i >> 6] >> (i & 63) & 1; }
template <int NW> static void words(Row& r, int a, int reach) {
  uint64_t v[NW];
  for (int w = 0; w < NW; ++w) v[w] = r[w];
  dilate_words(v, a, reach);
  for (int w = 0; w < NW; ++w) r[w] = v[w];
}
int main() {
  std::mt19937_64 rng(1);
  long n = 0;
  for (int S = 1; S <= 768; S = S < 200 ? S + 1 : S + 61) {
    const int nw = (S + 63) / 64;
    for (int a = 1; a <= S; a *= 2)
      for (int r = a; r <= S; r = S < 200 ? r + 1 : r + 1 + r / 9)
        for (int d = 0; d < 2; ++d) {  // sparse and half full
          Row in(nw, 0);
          for (int i = 0; i < S; ++i)
            if (rng() % (d ? 2 : 40) == 0) in[i >> 6] |= 1ull << (i & 63);
          const int So = (S - r) / a + 1;
          for (int kind = 0; kind < (nw <= 3 ? 2 : 1); ++kind) {
            Row got = in;
            if (kind == 0) dilate_row(got.data(), nw, a, r);
            else if (nw == 1) words<1>(got, a, r);
            else if (nw == 2) words<2>(got, a, r);
            else words<3>(got, a, r);
            for (int X = 0; X < So; ++X) {
              bool any = false;
              for (int i = a * X; i < a * X + r; ++i) any = any || bit(in, i);
              if (bit(got, X) != any) { printf("S %d a %d r %d kind %d bit %d\n", S, a, r, kind, X); return 1; }
            }
            ++n;
          }
        }
  }
  printf("%ld\n", n);
}
"""


def test_bitmap_rows_dilate_and_thin(tmp_path):
    """Grid sides up to 768 (three words a row in registers up to 192), every power-of-two step, every reach."""
    assert int(run_host(tmp_path, BIT_ROWS)) > 100000
