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

// Consecutive rows while they have at most kDenseArcs arcs and kDenseRows
// rows, and rows times the longest row stays within kDenseSpan; a longer row is
// cut into pieces of kDenseArcs arcs.  *nlong: rows so cut.
inline void dense_blocks(const std::vector<int64_t>& off, std::vector<DenseBlk>* out,
                         int32_t* nlong) {
  const int64_t n = (int64_t)off.size() - 1;
  *nlong = 0;
  out->reserve((size_t)(n / kDenseRows + 2 * (off[n] / kDenseArcs) + 16));
  for (int64_t v = 0; v < n;) {
    int64_t d = off[v + 1] - off[v];
    if (d > kDenseArcs) {
      const int32_t pieces = (int32_t)((d + kDenseArcs - 1) / kDenseArcs);
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
    // rows up to `end`, which the row limit and the longest row so far set
    const int64_t last = off[v] + kDenseArcs;
    int64_t w = v, top = 0, end = std::min<int64_t>(n, v + kDenseRows);
    for (; w < end && off[w + 1] <= last; w++) {
      d = off[w + 1] - off[w];
      if (d <= top) continue;
      const int64_t lim = v + kDenseSpan / d;
      if (w >= lim) break;
      top = d;
      end = std::min(end, lim);
    }
    const int64_t arcs = off[w] - off[v];
    if (arcs > 0)  // (isolated vertices take part in no round)
      out->push_back(DenseBlk{(int32_t)v, (int32_t)(w - v), -1, (int32_t)arcs, (long long)off[v]});
    v = w;
  }
}

}  // namespace plc
