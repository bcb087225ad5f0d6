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
    r = subprocess.run([str(exe)], timeout=120, stdout=subprocess.PIPE, text=True)
    assert r.returncode == 0, r.stdout
    return r.stdout


BIT_ROWS = r"""
#include "bit_rows.h"
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>
using namespace sscn;
typedef std::vector<uint64_t> Row;
static bool bit(const Row& r, int i) { return r[i >> 6] >> (i & 63) & 1; }
template <int NW> static void words(Row& r, int a, int reach, int n) {
  uint64_t v[NW];
  for (int w = 0; w < NW; ++w) v[w] = r[w];
  dilate_words(v, a, reach, n);
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
            else if (nw == 1) words<1>(got, a, r, So);
            else if (nw == 2) words<2>(got, a, r, So);
            else words<3>(got, a, r, So);
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


TILE_DEAL = r"""
#include "gemm_rules.h"
#include <cstdio>
#include <vector>
using namespace sscn;
int main() {
  const int limit = 2048;
  long n = 0;
  for (int cap = 1; cap <= 9000; cap = cap < 2200 ? cap + 1 : cap + 37)          // tiles at the row bound
    for (int nt = cap; nt >= 0; nt = cap < 400 ? nt - 1 : nt - 1 - (cap - nt) / 3)  // tiles of the rows present
      for (int by = 0; by < 2; ++by) {
        const int grid = deal_grid(cap, limit, by), plain = deal_grid(cap, limit, false);
        std::vector<char> seen(nt, 0);
        int most = 0;
        for (int b = 0; b < grid; ++b) {
          const TileDeal d = deal_tiles(nt, grid, b, by);
          if (d.step < 1) { printf("cap %d tiles %d dealt %d block %d: step %d\n", cap, nt, by, b, d.step); return 1; }
          int k = 0;
          for (int t = d.first; t < d.end; t += d.step, ++k)
            if (t < 0 || t >= nt || seen[t]++) { printf("cap %d tiles %d dealt %d block %d: tile %d\n", cap, nt, by, b, t); return 1; }
          most = k > most ? k : most;
        }
        for (int t = 0; t < nt; ++t)
          if (!seen[t]) { printf("cap %d tiles %d dealt %d: tile %d left out\n", cap, nt, by, t); return 1; }
        if (most > (nt + plain - 1) / plain) {
          printf("cap %d tiles %d dealt %d: %d tiles to a workgroup, %d in plain order\n", cap, nt, by, most, (nt + plain - 1) / plain);
          return 1;
        }
        ++n;
      }
  printf("%ld\n", n);
}
"""


def test_tiles_are_dealt_once_and_evenly(tmp_path):
    """Every tile once; no workgroup takes more tiles than with one tile after another in plain order."""
    assert int(run_host(tmp_path, TILE_DEAL)) > 100000


GEMM_MODES = r"""
#include "gemm_rules.h"
#include <cstdio>
int main() {
  for (int pool = 0; pool < 2; ++pool)
    for (int masked = 0; masked < 2; ++masked)
      for (int ac = -1; ac <= 4; ac += ac < 0 ? 1 : 4)  // no pooling backward, or its window count
        for (int ks = 1; ks < 4; ++ks)
          printf("%d %d %d %d %d\n", pool, masked, ac, ks, sscn::gemm_mode(pool, masked, ac >= 0, ac < 0 ? 0 : ac, ks));
}
"""


def test_split_k_launches_are_plain(tmp_path):
    """The masked instantiation reads the layer below's tile for its own store; with K split only the
    reduce stores."""
    for line in run_host(tmp_path, GEMM_MODES).splitlines():
        pool, masked, ac, ks, mode = map(int, line.split())
        want = -2 if pool else -3 if masked and ks == 1 else ac
        assert mode == want, line


CHUNKS = r"""
#include "gemm_rules.h"
#include <cstdio>
int main() {
  const long long at[][3] = {{108, 57, 32}, {310, 158, 83}, {338, 210, 147}, {512, 300, 160}, {513, 300, 160}, {686, 388, 259},
                             {1346, 691, 362}, {1400, 700, 370}, {1402, 701, 370}, {1416, 769, 428}, {1273, 766, 384}};
  for (auto& t : at)
    for (int div = 1; div <= 4; div *= 2) {  // planned lengths: the last `levels` of (quarter, half, standard)
      const int skip = div == 4 ? 0 : div == 2 ? 1 : 2;
      long tiles[3] = {0, 0, 0};
      for (int i = 0; i + skip < 3; ++i) tiles[i] = t[i + skip];
      printf("%lld %lld %d %d\n", t[0], t[1], div, sscn::chunk_multiple(div, tiles));
    }
}
"""


def test_chunks_are_as_short_as_the_passes_own_tiles_allow(tmp_path):
    """A quarter of the standard length with at most 512 tiles, else a half with at most 700, else the
    standard one; never shorter than planned."""
    for line in run_host(tmp_path, CHUNKS).splitlines():
        quarter, half, div, got = map(int, line.split())
        want = 4 if quarter <= 512 and div == 4 else 2 if half <= 700 and div >= 2 else 1  # parts of the standard length
        assert div // got == want and div % got == 0, line
