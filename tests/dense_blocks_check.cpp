// dense_blocks and dense_blocks_most on the CPU: the blocks cover every arc
// once within their limits and are as long as those allow, a lane of the dense round sums fewer than 128
// products of a row, and no graph has more blocks than dense_blocks_most, also
// those whose blocks end as early as each limit allows.  Prints
// "n arcs most" lines for test_dense_blocks.py, which builds and runs it.
#include <cstdio>
#include <random>
#include <vector>

#include "../paper_1604_07515_amd/csrc/dense_blocks.h"

#define CHECK(c)                                                        \
  do {                                                                  \
    if (!(c)) {                                                         \
      std::fprintf(stderr, "check failed line %d: %s\n", __LINE__, #c); \
      return 1;                                                         \
    }                                                                   \
  } while (0)

static int check(const std::vector<int32_t>& deg) {
  const int64_t n = (int64_t)deg.size();
  std::vector<int64_t> off((size_t)n + 1, 0);
  for (int64_t v = 0; v < n; v++) off[v + 1] = off[v] + deg[v];
  std::vector<plc::DenseBlk> blk;
  int32_t nlong = -1;
  plc::dense_blocks(off, deg.data(), &blk, &nlong);
  int64_t row = 0, lids = 0, at = 0;
  for (size_t i = 0; i < blk.size(); i++) {
    const plc::DenseBlk& b = blk[i];
    for (; row < b.row; row++) CHECK(deg[row] == 0);
    CHECK(b.first == at && b.len >= 1 && b.len <= plc::kDenseArcs);
    at += b.len;
    if (b.lid >= 0) {
      const int32_t d = deg[b.row];
      CHECK(d > plc::kDenseArcs && b.lid == lids);
      CHECK(b.nrows == (d + plc::kDenseArcs - 1) / plc::kDenseArcs);
      if (at == off[b.row + 1]) {
        lids++;
        row = b.row + 1;
      }
      continue;
    }
    CHECK(b.row == row && b.nrows >= 1 && b.nrows <= plc::kDenseRows && at == off[row + b.nrows]);
    int32_t top = 0;
    for (int r = 0; r < b.nrows; r++) top = std::max(top, deg[b.row + r]);
    CHECK((int64_t)top * b.nrows <= plc::kDenseSpan);
    if (row + b.nrows < n) {  // it ends only where the next row would break a limit
      const int32_t d = deg[row + b.nrows];
      CHECK(b.nrows == plc::kDenseRows || b.len + d > plc::kDenseArcs ||
            (int64_t)(b.nrows + 1) * std::max(top, d) > plc::kDenseSpan);
    }
    int lanes = 1;  // of 256 threads per row, a power of two, at most a wave
    while (2 * lanes * b.nrows <= 256 && lanes < 64) lanes *= 2;
    CHECK((top + lanes - 1) / lanes < 2 * plc::kDenseSpan / 256);
    row += b.nrows;
  }
  for (; row < n; row++) CHECK(deg[row] == 0);
  CHECK(at == off[n] && lids == nlong);
  CHECK((int64_t)blk.size() <= plc::dense_blocks_most(n, off[n]));
  std::printf("%lld %lld %lld\n", (long long)n, (long long)off[n],
              (long long)plc::dense_blocks_most(n, off[n]));
  return 0;
}

int main() {
  std::mt19937_64 rng(5);
  for (int n : {1, 15, 16, 17, 255, 256, 257, 4097, 50000}) {
    for (int kind = 0; kind < 12; kind++) {
      std::vector<int32_t> d((size_t)n);
      for (int v = 0; v < n; v++) {
        const int r = (int)(rng() % 1000);
        switch (kind) {
          case 0: d[v] = 0; break;
          case 1: d[v] = 1; break;
          case 2: d[v] = 2049; break;                       // two pieces, the second of one arc
          case 3: d[v] = v % 2 ? 2049 : 1; break;           // and a short block before each
          case 4: d[v] = v % 2 ? 2048 : 1; break;           // ends for its arcs
          case 5: d[v] = v % 129 ? 1 : 127; break;          // one lane a row, 127 products
          case 6: d[v] = v % 256 ? 0 : 65; break;           // ends for rows times longest row
          case 7: d[v] = v % 16 ? 0 : 1025; break;
          case 8: d[v] = v % 65 ? 1 : 256; break;
          case 9: d[v] = r % 40; break;
          case 10: d[v] = r < 990 ? r % 4 : 100 * (r - 985); break;
          default: d[v] = r < 500 ? 0 : (int)(rng() % 4200); break;
        }
      }
      if (check(d)) {
        std::fprintf(stderr, "kind %d n %d\n", kind, n);
        return 1;
      }
    }
  }
  std::puts("blocks ok");
  return 0;
}
