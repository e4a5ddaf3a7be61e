// dense_blocks.h -- the rows of a graph cut into the blocks of the dense round
// (host).
#pragma once
#include <algorithm>
#include <cmath>
#include <cstddef>
#include <cstdint>
#include <vector>

namespace plc {

constexpr int kDenseRows = 256;    // rows of a block, at most
constexpr int kDenseArcs = 2048;   // its arcs, at most
constexpr int kDenseSpan = 16384;  // its rows times its longest row, at most

// One block of the dense round: nrows consecutive rows from row on (at most
// kDenseRows, kDenseArcs arcs), or, with lid >= 0, one piece of the arcs of a
// row longer than kDenseArcs (nrows pieces in all).
struct alignas(32) DenseBlk {
  int32_t row, nrows, lid, len;
  long long first;  // first arc and number of arcs
};

// Blocks of any graph of n vertices and this many arcs, at most.  A row longer
// than kDenseArcs has at most twice its arcs over kDenseArcs pieces, and ends
// the block before it; a block that ends for its arcs has, with the row after
// it, more than kDenseArcs; one that ends for kDenseSpan with k rows has, with
// the row after it, one of more than kDenseSpan / (k + 1) arcs (a row counts
// for two blocks at most: the Cauchy-Schwarz inequality over those and k + 1).
inline int64_t dense_blocks_most(int64_t n, int64_t arcs) {
  const double x = (double)arcs / (kDenseSpan / 2);
  return 3 * arcs / kDenseArcs + n / kDenseRows + (int64_t)(x + std::sqrt(x * (double)n)) + 4;
}

// Consecutive rows while they have at most kDenseArcs arcs and kDenseRows rows,
// and rows times the longest row stays within kDenseSpan; a longer row is cut
// into pieces of kDenseArcs arcs.  *nlong: rows so cut.
//
// Every graph load pays for it.  Rows times longest row only grows along a
// block, so whole chunks are tested by their longest row and only the chunk in
// which the block ends row by row: 0.25 ms on R-MAT 2^20 (31 M arcs, loaded in
// 13.8 ms), 0.50 row by row throughout.
inline void dense_blocks(const std::vector<int64_t>& off, const int32_t* deg,
                         std::vector<DenseBlk>* out, int32_t* nlong) {
  constexpr int kChunk = 16;
  const int64_t n = (int64_t)off.size() - 1;
  *nlong = 0;
  out->reserve((size_t)(n / kDenseRows + 2 * (off[n] / kDenseArcs) + 16));
  for (int64_t v = 0; v < n;) {
    const int32_t d = deg[v];
    if (d > kDenseArcs) {
      const int32_t pieces = (int32_t)(((int64_t)d + kDenseArcs - 1) / kDenseArcs);
      for (int32_t k = 0; k < pieces; k++) {
        const int64_t e = (int64_t)k * kDenseArcs;
        out->push_back(DenseBlk{(int32_t)v, pieces, *nlong,
                                (int32_t)std::min<int64_t>(kDenseArcs, d - e),
                                (long long)(off[v] + e)});
      }
      (*nlong)++;
      v++;
      continue;
    }
    const int64_t end = std::min<int64_t>(n, v + kDenseRows), last = off[v] + kDenseArcs;
    int64_t w = v;
    int64_t top = 0;
    for (; w + kChunk <= end && off[w + kChunk] <= last; w += kChunk) {
      int32_t m = 0;
      for (int k = 0; k < kChunk; k++) m = std::max(m, deg[w + k]);
      if ((w + kChunk - v) * std::max<int64_t>(top, m) > kDenseSpan) break;
      top = std::max<int64_t>(top, m);
    }
    for (; w < end && off[w + 1] <= last; w++) {
      top = std::max<int64_t>(top, deg[w]);
      if ((w + 1 - v) * top > kDenseSpan) break;
    }
    const int64_t arcs = off[w] - off[v];
    if (arcs > 0)  // (isolated vertices take part in no round)
      out->push_back(DenseBlk{(int32_t)v, (int32_t)(w - v), -1, (int32_t)arcs, (long long)off[v]});
    v = w;
  }
}

}  // namespace plc
