// Word-parallel transforms of one row of an occupancy bitmap: bit X of the result
// is set when any of bits [a X, a X + r) of the row is (a a power of two; bits past
// the row's end read as zero, and result bits past its own end are the caller's to
// mask).  The dilation doubles its reach (log2 r shifts of the whole row), then
// every a-th bit is kept (log2 a rounds of packing the even bits): a few dozen
// operations a word, where a test of each output bit's range takes a whole row of
// tests.  constexpr, so the device code and a host program run the same text.
#pragma once

#include <stdint.h>

namespace sscn {

// Bits 0, 2, 4, .. of v, packed into 32 bits.
constexpr inline uint64_t even_bits(uint64_t v) {
  v &= 0x5555555555555555ull;
  v = (v | (v >> 1)) & 0x3333333333333333ull;
  v = (v | (v >> 2)) & 0x0f0f0f0f0f0f0f0full;
  v = (v | (v >> 4)) & 0x00ff00ff00ff00ffull;
  v = (v | (v >> 8)) & 0x0000ffff0000ffffull;
  return (v | (v >> 16)) & 0xffffffffull;
}

// A row of nw words in memory, in place.
constexpr inline void dilate_row(uint64_t* row, int nw, int a, int r) {
  for (int len = 1; len < r;) {
    const int sh = len < r - len ? len : r - len, ws = sh >> 6, bs = sh & 63;
    for (int w = 0; w < nw; ++w) {  // words >= w only: in place
      const uint64_t lo = w + ws < nw ? row[w + ws] : 0ull, hi = w + ws + 1 < nw ? row[w + ws + 1] : 0ull;
      row[w] |= bs ? (lo >> bs) | (hi << (64 - bs)) : lo;
    }
    len += sh;
  }
  for (int st = a; st > 1; st >>= 1) {
    for (int w = 0; w < (nw + 1) / 2; ++w) {
      const uint64_t lo = row[2 * w], hi = 2 * w + 1 < nw ? row[2 * w + 1] : 0ull;
      row[w] = even_bits(lo) | (even_bits(hi) << 32);
    }
    nw = (nw + 1) / 2;
  }
}

// A row of NW <= 3 words in registers, r <= 64 NW: no shift is longer than a word
// (they go 1, 2, .. 64, and the last covers what is left of r).  In the row buffer
// each word of each round was a dependent chain through LDS, which cost more than
// the per-bit tests on grids of up to 128 columns: the whole bitmap launch at
// batch 1600, 96 x 96 grids, 36.8 us by tests, 37.9 in LDS, 33.0 like this; 24 x 24
// 17.0, 18.5, 15.6; batch 64, 192 x 192 25.9, 12.3, 10.8.
template <int NW>
constexpr inline void dilate_words(uint64_t (&row)[NW], int a, int r) {
  static_assert(NW >= 1 && NW <= 3, "no shift above 64");
  for (int len = 1; len < r;) {
    const int sh = len < r - len ? len : r - len;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const uint64_t hi = w + 1 < NW ? row[w + 1 < NW ? w + 1 : w] : 0ull;
      row[w] |= sh < 64 ? (row[w] >> sh) | (hi << (64 - sh)) : hi;
    }
    len += sh;
  }
  int nw = NW;
  for (int st = a; st > 1; st >>= 1) {
#pragma unroll
    for (int w = 0; w < (NW + 1) / 2; ++w) {
      if (2 * w >= nw) continue;
      const uint64_t hi = 2 * w + 1 < NW ? row[2 * w + 1 < NW ? 2 * w + 1 : w] : 0ull;
      row[w] = even_bits(row[2 * w]) | (2 * w + 1 < nw ? even_bits(hi) << 32 : 0ull);
    }
    nw = (nw + 1) / 2;
  }
}

}  // namespace sscn
