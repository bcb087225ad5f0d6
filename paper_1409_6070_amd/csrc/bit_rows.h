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

// A row of NW <= 3 words in registers, r <= 64 NW, of which n result bits are wanted:
// no shift is longer than a word (they go 1, 2, .. 64, and the last covers what is
// left of r).  Up to eight bits are picked one by one, about six operations each
// against thirty for each round of packing a word.  (In the row buffer each word of
// each round was a dependent chain through LDS.  The whole bitmap launch by per-bit
// tests / in the row buffer / in registers: 96 x 96 grids at batch 1600 36.7 / 37.8 /
// 33.3 us, at batch 100 10.1 / 9.7 / 8.3; 192 x 192 at batch 64 25.9 / 12.4 / 10.9;
// 48 x 48 at batch 8 7.0 / 7.3 / 6.2; 12 x 12 at batch 2 4.8 / 6.2 / 5.6.)
template <int NW>
constexpr inline void dilate_words(uint64_t (&row)[NW], int a, int r, int n) {
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
  if (a > 1 && n <= 8) {
    uint64_t bits = 0;
    for (int X = 0; X < n; ++X) {
      const int at = a * X;
      uint64_t v = row[0];
#pragma unroll
      for (int w = 1; w < NW; ++w) v = at >= 64 * w ? row[w] : v;
      bits |= ((v >> (at & 63)) & 1ull) << X;
    }
    row[0] = bits;
#pragma unroll
    for (int w = 1; w < NW; ++w) row[w] = 0ull;
    return;
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
