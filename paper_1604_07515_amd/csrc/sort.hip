// sort.hip -- device sort of the sweep order (Sec. 3.1: the support sorted
// by non-increasing p/d).  Elements are (seg, key, id) triples ordered
// lexicographically ascending: seg separates the supports of different
// queries, key is the bit-inverted IEEE pattern of the positive ratio p/d
// (ascending key = non-increasing ratio) and id breaks ties (ascending id).
//
// Merge sort: one launch sorts 4096-element tiles in LDS (each of 512
// threads sorts 8 elements in registers with a bitonic network, then nine
// rounds of merge-path merges in LDS double the sorted runs up to the tile),
// then
// each merge pass doubles the sorted run length.  A pass produces
// 1024-element output tiles; the two split points of a tile on the merge
// path are found by a cooperative 128-ary search (a few rounds of parallel
// global loads, each resolved with wave ballots instead of a serial binary
// search), the inputs are staged in LDS and every thread merges four
// outputs.  The element count lives in
// device memory; passes whose run length already covers it return at once,
// so the whole sequence is queued without a host round trip.
//
// Small counts (a bound of at most kRankMaxCount elements known when the
// sort is queued) sort tiles of 1024 instead, so that a support of a few
// thousand vertices is on several CUs, and replace the merge passes with one
// launch: each element's place is its position in its own tile plus its
// count in every other tile, found by binary searches in tiles held in LDS,
// and the last of those additions places it.  Many segments of at most so
// many elements each (launch_seg_sort) are sorted the same way, every segment
// within its own range of the buffer.
//
// The first launch can carry a side job (SortArgs::side_ids) for its
// workgroups that hold no tile: with supports of a few tiles most of the
// launch's workgroups would otherwise only exit.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "device_util.h"
#include "sort.h"

namespace plc {

constexpr int kSortBlk = 256;
constexpr int kTileS = 1024;        // elements per merge-pass output tile
constexpr int kPerThr = kTileS / kSortBlk;
constexpr int kBSBlk = 512;         // threads of the block sort
constexpr int kBT = 8;              // elements per thread in the block sort
constexpr int kTileB = kBSBlk * kBT;    // elements per block-sort tile

// The largest element: pads a tile past the element count.
constexpr SortElem kMaxElem = {~0ull, INT32_MAX, INT32_MAX};

// LDS index of element i of a block-sort tile: one spare slot after every
// kBT elements, so the kBT-element rows of consecutive threads start on
// different banks.
__device__ __forceinline__ int lds_pad(int i) { return i + i / kBT; }

// The comparison and the selects take whole elements by value and use no
// short-circuit operators: every field of both operands is loaded up front
// (one 16-byte load each) instead of one dependent load per field compared.
__device__ __forceinline__ bool elem_lt(const SortElem a, const SortElem b) {
  const bool seg_lt = a.seg < b.seg, seg_eq = a.seg == b.seg;
  const bool key_lt = a.key < b.key, key_eq = a.key == b.key;
  return seg_lt | (seg_eq & (key_lt | (key_eq & (a.id < b.id))));
}

__device__ __forceinline__ SortElem elem_sel(bool c, const SortElem a, const SortElem b) {
  SortElem r;
  r.key = c ? a.key : b.key;
  r.id = c ? a.id : b.id;
  r.seg = c ? a.seg : b.seg;
  return r;
}

// Element i of a sorted run in LDS (index through idx), or the largest
// element once i reaches the run's length: the load uses a clamped index,
// so it stays an LDS load and never needs the constant from memory.
template <typename F>
__device__ __forceinline__ SortElem run_head(const SortElem* sh, F idx, int i, int len) {
  const SortElem v = sh[idx(i < len ? i : len - 1)];
  return elem_sel(i < len, v, kMaxElem);
}

__device__ __forceinline__ bool sort_enabled(const SortArgs& s) {
  return s.active == nullptr || *s.active == s.active_value;
}

// Compare-exchange: afterwards a <= b when up, a >= b otherwise.
__device__ __forceinline__ void cswap(SortElem& a, SortElem& b, bool up) {
  const bool sw = elem_lt(b, a) == up;
  const SortElem lo = elem_sel(sw, b, a);
  const SortElem hi = elem_sel(sw, a, b);
  a = lo;
  b = hi;
}

constexpr int kSideItems = 4;                    // side-job entries per thread and step
constexpr int kSideGrid = 512;                   // block-sort workgroups when a side job rides along

// The first launch's side job (SortArgs::side_ids), in steps of
// NT * kSideItems ids per workgroup of NT threads: the workgroups are renumbered so that those
// holding no tile take the first steps; the ones that sorted a tile join
// only when there are more steps than workgroups without one.  Each step
// places its nonzeros with one workgroup scan and one global atomic.
template <int NT>
__device__ void side_job(const SortArgs& s, int ntiles) {
  constexpr int kSideStep = NT * kSideItems;
  long long T = *s.side_count;
  if (T > s.side_out_cap) T = s.side_out_cap;
  if (T <= 0) return;
  __shared__ long long sh[NT / 64 + 1];
  __shared__ long long s_base;
  const int G = gridDim.x;
  const int busy = ntiles < G ? ntiles : G;
  const int w = ((int)blockIdx.x - busy + G) % G;
  const int t = threadIdx.x;
  for (long long base = (long long)w * kSideStep; base < T; base += (long long)G * kSideStep) {
    int32_t v[kSideItems];
    double x[kSideItems];
#pragma unroll
    for (int k = 0; k < kSideItems; k++) {
      const long long i = base + k * NT + t;
      v[k] = i < T ? s.side_ids[i] : -1;
    }
#pragma unroll
    for (int k = 0; k < kSideItems; k++)
      x[k] = v[k] >= 0 ? s.side_val[(long long)v[k] * s.side_stride] : 0.0;
    long long cnt = 0;
#pragma unroll
    for (int k = 0; k < kSideItems; k++) {
      if (v[k] >= 0) s.side_val[(long long)v[k] * s.side_stride] = 0.0;
      cnt += x[k] != 0.0;
    }
    long long tot;
    const long long off = block_excl_scan<NT>(cnt, &tot, sh);
    if (t == 0) s_base = tot > 0 ? atomicAdd(s.side_out_cnt, (int32_t)tot) : 0;
    __syncthreads();
    long long slot = s_base + off;
#pragma unroll
    for (int k = 0; k < kSideItems; k++) {
      if (x[k] != 0.0) {
        if (slot < s.side_out_cap) {
          s.side_out_id[slot] = v[k];
          s.side_out_val[slot] = x[k];
        } else {
          *s.side_fault = 1;
        }
        slot++;
      }
    }
    __syncthreads();
  }
}

// Where the sorted elements end up follows from the count, so nothing of the
// sort counts its workgroups (512 additions to one word outlast the merging
// of 30,000 elements).
__global__ __launch_bounds__(kBSBlk) void k_block_sort(SortArgs s) {
  const int N = *s.count;
  if (!sort_enabled(s)) return;
  SortElem* buf = s.buf[0];
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    int flip = 0;
    for (long long L = kTileB; L < N; L <<= 1) flip ^= 1;
    *s.flip = flip;
  }
  __shared__ SortElem sh[kTileB + kTileB / kBT];
  const int ntiles = (N + kTileB - 1) / kTileB;
  const int t = threadIdx.x;
  for (int tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
    const int base = tile * kTileB;
    // coalesced load (element k*256 + t), padded past N with the largest element
#pragma unroll
    for (int k = 0; k < kBT; k++) {
      const int i = k * kBSBlk + t;
      const int gi = base + i < N ? base + i : N - 1;
      sh[lds_pad(i)] = elem_sel(base + i < N, buf[gi], kMaxElem);
    }
    __syncthreads();
    // elements kBT*t .. kBT*t + kBT - 1, sorted in registers (bitonic network)
    SortElem x[kBT];
#pragma unroll
    for (int k = 0; k < kBT; k++) x[k] = sh[lds_pad(t * kBT + k)];
#pragma unroll
    for (int k = 2; k <= kBT; k <<= 1) {
#pragma unroll
      for (int j = k >> 1; j > 0; j >>= 1) {
#pragma unroll
        for (int i = 0; i < kBT; i++) {
          const int l = i ^ j;
          if (l > i) cswap(x[i], x[l], (i & k) == 0);
        }
      }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kBT; k++) sh[lds_pad(t * kBT + k)] = x[k];
    __syncthreads();
    // merge runs of L into runs of 2L; thread t produces outputs
    // [kBT*t, kBT*t + kBT) of the tile, i.e. diagonal d of its pair of runs
    for (int L = kBT; L < kTileB; L <<= 1) {
      const int o = t * kBT;
      const int pb = (o / (2 * L)) * (2 * L);
      const int d = o - pb;
      const int A = pb, B = pb + L;  // run starts (tile positions)
      int lo = d - L > 0 ? d - L : 0;
      int hi = d < L ? d : L;
      while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        const SortElem b = sh[lds_pad(B + d - 1 - mid)];
        const SortElem a = sh[lds_pad(A + mid)];
        if (elem_lt(b, a)) hi = mid; else lo = mid + 1;
      }
      // the two run heads stay in registers; an exhausted run shows the
      // largest element, equal to the tile padding, so either choice
      // between the two then outputs the same value
      int ia = lo, ib = d - lo;
      SortElem ha = run_head(sh, [&](int i) { return lds_pad(A + i); }, ia, L);
      SortElem hb = run_head(sh, [&](int i) { return lds_pad(B + i); }, ib, L);
#pragma unroll
      for (int k = 0; k < kBT; k++) {
        const bool ta = !elem_lt(hb, ha);
        x[k] = elem_sel(ta, ha, hb);
        ia += ta;
        ib += !ta;
        // one load: the next head of the run just taken
        const int r0 = ta ? A : B;
        const int ri = ta ? ia : ib;
        const SortElem nx = run_head(sh, [&](int i) { return lds_pad(r0 + i); }, ri, L);
        ha = elem_sel(ta, nx, ha);
        hb = elem_sel(ta, hb, nx);
      }
      __syncthreads();
#pragma unroll
      for (int k = 0; k < kBT; k++) sh[lds_pad(o + k)] = x[k];
      __syncthreads();
    }
#pragma unroll
    for (int k = 0; k < kBT; k++) {
      const int i = k * kBSBlk + t;
      if (base + i < N) {
        buf[base + i] = sh[lds_pad(i)];
      }
    }
    __syncthreads();
  }
  if (s.side_ids != nullptr) side_job<kBSBlk>(s, ntiles);
}

// ------------------------------------------------------ small-count path

constexpr int kTileR = 1024;                           // elements per tile
constexpr int kTSBlk = 512;                            // threads of the tile sort
constexpr int kRankBlk = 512;                          // threads of the rank merge
constexpr int kRankTiles = 4;                          // tiles a workgroup holds in LDS
constexpr int kRankSpan = kRankTiles * kTileR;
constexpr int kRankGrid = 512;                         // its workgroups, at most
static_assert(kRankMaxCount % kRankSpan == 0, "whole groups of tiles");

// An element with its key turned back into the ratio: the searches compare
// millions of pairs, and two double comparisons (full rate) take the place of
// two 64-bit integer ones.  Ratios are positive; the padding past the count
// has ratio -1 and an id of its own, so that no two elements are equal.
struct __align__(16) RankElem {
  double ratio;
  int32_t id, seg;
};
__device__ __forceinline__ RankElem rank_elem(const SortElem e) {
  return RankElem{__longlong_as_double((long long)~e.key), e.id, e.seg};
}
// No segment in it: the elements compared are of one segment.
__device__ __forceinline__ bool rank_lt(const RankElem a, const RankElem b) {
  return (a.ratio > b.ratio) | ((a.ratio == b.ratio) & (a.id < b.id));
}

// Sorts src[0 .. len) into dst (which may be src) and writes every element's
// place to rank: pairs, then runs of L merge into runs of 2 L by rank: an
// element's place is its position plus its count in the sibling run, a
// branch-free binary search in LDS (a merge-path round of the block sort
// takes as many LDS round trips, and then one per output).
__device__ void tile_sort(const SortElem* src, SortElem* dst, unsigned long long* rank, int len,
                          RankElem (*sh)[kTileR]) {
  const int t = threadIdx.x;
  static_assert(kTileR == 2 * kTSBlk, "two elements per thread");
  {
    const int i = 2 * t;
    RankElem a{-1.0, i, INT32_MAX}, b{-1.0, i + 1, INT32_MAX};
    if (i < len) a = rank_elem(src[i]);
    if (i + 1 < len) b = rank_elem(src[i + 1]);
    const bool sw = rank_lt(b, a);
    sh[0][sw ? i + 1 : i] = a;
    sh[0][sw ? i : i + 1] = b;
  }
  __syncthreads();
  int cur = 0;
  for (int L = 2; L < len; L <<= 1, cur ^= 1) {
    const RankElem* in = sh[cur];
    RankElem* out = sh[cur ^ 1];
    const RankElem x0 = in[t], x1 = in[t + kTSBlk];
    const RankElem* s0 = in + ((t & ~(L - 1)) ^ L);
    const RankElem* s1 = in + (((t + kTSBlk) & ~(L - 1)) ^ L);
    int c0 = 0, c1 = 0;
    for (int h = L >> 1; h > 0; h >>= 1) {
      const RankElem y0 = s0[c0 + h - 1], y1 = s1[c1 + h - 1];
      c0 += rank_lt(y0, x0) ? h : 0;
      c1 += rank_lt(y1, x1) ? h : 0;
    }
    c0 += rank_lt(s0[c0], x0) ? 1 : 0;
    c1 += rank_lt(s1[c1], x1) ? 1 : 0;
    out[(t & ~(2 * L - 1)) + (t & (L - 1)) + c0] = x0;
    out[((t + kTSBlk) & ~(2 * L - 1)) + (t & (L - 1)) + c1] = x1;
    __syncthreads();
  }
  static_assert((kTSBlk & (kTSBlk - 1)) == 0, "t and t + kTSBlk agree below a run's length");
#pragma unroll
  for (int k = 0; k < 2; k++) {
    const int i = k * kTSBlk + t;
    if (i < len) {
      const RankElem e = sh[cur][i];
      dst[i] = SortElem{~(unsigned long long)__double_as_longlong(e.ratio), e.id, e.seg};
      rank[i] = (unsigned long long)i;
    }
  }
  __syncthreads();
}

// Tiles of one segment.  On R-MAT 2^22 queries (30,000 elements, the side
// job beside it) 13.7 us where the block sort of 4096-element tiles took 32,
// which it took for 100 elements too (now 3.9).
__global__ __launch_bounds__(kTSBlk) void k_tile_sort(SortArgs s) {
  const int N = *s.count;
  if (!sort_enabled(s)) return;
  SortElem* buf = s.buf[0];
  if (blockIdx.x == 0 && threadIdx.x == 0) *s.flip = N > kTileR;
  __shared__ RankElem sh[2][kTileR];
  const int ntiles = (N + kTileR - 1) / kTileR;
  for (int tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
    const int base = tile * kTileR;
    tile_sort(buf + base, buf + base, s.rank + base, N - base < kTileR ? N - base : kTileR, sh);
  }
  if (s.side_ids != nullptr) side_job<kTSBlk>(s, ntiles);
}

// How many elements of the len in sh (sorted tiles of kTileR) come before x,
// tile `own` left out: one search per tile, in flight together.
__device__ __forceinline__ int rank_in(const RankElem* sh, int len, int own, const RankElem x) {
  int n[kRankTiles], c[kRankTiles];
#pragma unroll
  for (int k = 0; k < kRankTiles; k++) {
    const int r = len - k * kTileR;
    n[k] = k == own ? 0 : r < kTileR ? r : kTileR;  // (<= 0: nothing to count)
    c[k] = 0;
  }
  for (int h = kTileR; h > 0; h >>= 1) {
#pragma unroll
    for (int k = 0; k < kRankTiles; k++) {
      const int at = c[k] + h - 1;
      const RankElem y = sh[k * kTileR + (at < n[k] ? at : 0)];
      c[k] += (at < n[k]) & rank_lt(y, x) ? h : 0;
    }
  }
  int lo = 0;
#pragma unroll
  for (int k = 0; k < kRankTiles; k++) lo += c[k];
  return lo;
}

// Adds group's count lo to element q's rank and places it at dst once the
// counts of all groups are in (q0: its position in its own tile).
__device__ __forceinline__ void rank_add(SortElem* dst, unsigned long long* rank, int groups,
                                         int q0, int lo, const SortElem e) {
  if (groups == 1) {
    dst[q0 + lo] = e;
    return;
  }
  const unsigned long long old = atomicAdd(rank, (1ull << 32) | (unsigned long long)lo);
  if ((int)(old >> 32) == groups - 1) dst[(long long)(old & 0xffffffffull) + lo] = e;
}

// Places every element of the sorted tiles at its rank in the whole order.
// Workgroup (j, g) of the per workgroups of tile group j holds the group's
// kRankTiles tiles in LDS and takes every per-th element: each lane counts
// the elements of those tiles (its own left out) that come before its
// element, one search per tile in flight together, and adds the count to the
// element's rank word (set by the tile sort to its position in its own tile),
// whose upper half counts the groups; the addition that completes them
// writes the element out.
__global__ __launch_bounds__(kRankBlk) void k_rank_merge(SortArgs s, int groups_max, int per) {
  const int N = *s.count;
  if (!sort_enabled(s)) return;
  if (N <= kTileR) return;
  const int groups = (N + kRankSpan - 1) / kRankSpan;
  const SortElem* src = s.buf[0];
  __shared__ RankElem sh[kRankSpan];
  const int g = blockIdx.x % per;
  for (int j = blockIdx.x / per; j < groups; j += groups_max) {
    const int base = j * kRankSpan;
    const int len = N - base < kRankSpan ? N - base : kRankSpan;
    __syncthreads();
    for (int x = threadIdx.x; x < len; x += kRankBlk) sh[x] = rank_elem(src[base + x]);
    __syncthreads();
    for (int q = g * kRankBlk + threadIdx.x; q < N; q += per * kRankBlk) {
      const SortElem e = src[q];
      const int lo = rank_in(sh, len, q / kTileR - j * kRankTiles, rank_elem(e));
      rank_add(s.buf[1], s.rank + q, groups, q & (kTileR - 1), lo, e);
    }
  }
}

static void rank_sort(hipStream_t st, const SortArgs& s, int64_t max_count) {
  // a side job takes the workgroups without a tile: two per CU keep the
  // gather from outlasting the sort
  const int tiles = (int)((max_count + kTileR - 1) / kTileR);
  const int grid = s.side_ids != nullptr ? kSideGrid : tiles;
  hipLaunchKernelGGL(k_tile_sort, dim3(grid), dim3(kTSBlk), 0, st, s);
  if (tiles <= 1) return;
  // one element per thread while that keeps to kRankGrid workgroups
  const int groups = (int)((max_count + kRankSpan - 1) / kRankSpan);
  const int want = (int)((max_count + kRankBlk - 1) / kRankBlk);
  const int most = kRankGrid / groups;
  const int per = want < most ? want : most;
  hipLaunchKernelGGL(k_rank_merge, dim3(groups * per), dim3(kRankBlk), 0, st, s, groups, per);
}

// ------------------------------------------------------ many small segments

// The segment of tile (or merge item) x: the last one that starts at or
// before it.  first[] holds every segment's first tile (item); a segment
// without any shares its number with the next one and is passed over.
__device__ __forceinline__ int seg_at(const int32_t* first, int nseg, int x) {
  int lo = 0, hi = nseg - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (first[mid] <= x) lo = mid; else hi = mid - 1;
  }
  return lo;
}

__device__ __forceinline__ const SortSeg& seg_rec(const SegSort& g, int j) {
  return *reinterpret_cast<const SortSeg*>(g.seg + (size_t)j * g.stride);
}

// A sweep's segments are sorted each by itself: their ranges in the buffer are
// known, so the passes that a sort of the whole buffer needs for the segments'
// number are not made.  Sweep of 256 queries of R-MAT 2^22 (1.2 M elements):
// 142 us with the merge where block sort and merge passes took 310.
__global__ __launch_bounds__(kTSBlk) void k_seg_tile_sort(SortArgs s, SegSort g) {
  __shared__ RankElem sh[2][kTileR];
  __shared__ int32_t first[kMaxSortSegs];
  if (blockIdx.x == 0 && threadIdx.x == 0) *s.flip = 1;
  for (int j = threadIdx.x; j < g.nseg; j += kTSBlk) first[j] = seg_rec(g, j).tile0;
  __syncthreads();
  for (int tile = blockIdx.x; tile < g.tiles; tile += gridDim.x) {
    const int j = seg_at(first, g.nseg, tile);
    const SortSeg sg = seg_rec(g, j);
    const int at = (tile - sg.tile0) * kTileR;
    const long long base = sg.elem_off + at;
    const int len = sg.n_elem - at < kTileR ? sg.n_elem - at : kTileR;
    // a segment of one tile is done, and goes where the others will be
    tile_sort(s.buf[0] + base, s.buf[sg.n_elem <= kTileR] + base, s.rank + base, len, sh);
  }
}

// Item (tile i, group j) of a segment: the elements of its tile i against its
// tile group j, as in k_rank_merge.
__global__ __launch_bounds__(kRankBlk) void k_seg_merge(SortArgs s, SegSort g) {
  __shared__ RankElem sh[kRankSpan];
  __shared__ int32_t first[kMaxSortSegs];
  for (int j = threadIdx.x; j < g.nseg; j += kRankBlk) first[j] = seg_rec(g, j).item0;
  for (int item = blockIdx.x; item < g.items; item += gridDim.x) {
    __syncthreads();
    const SortSeg sg = seg_rec(g, seg_at(first, g.nseg, item));
    const int n = sg.n_elem, r = item - sg.item0;
    const int tiles = (n + kTileR - 1) / kTileR;
    const int groups = (tiles + kRankTiles - 1) / kRankTiles;
    const int i = r / groups, j = r % groups;
    const SortElem* src = s.buf[0] + sg.elem_off;
    const int base = j * kRankSpan;
    const int len = n - base < kRankSpan ? n - base : kRankSpan;
    for (int x = threadIdx.x; x < len; x += kRankBlk) sh[x] = rank_elem(src[base + x]);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kTileR / kRankBlk; k++) {
      const int q0 = k * kRankBlk + threadIdx.x, q = i * kTileR + q0;
      if (q >= n) continue;
      const SortElem e = src[q];
      const int lo = rank_in(sh, len, i - j * kRankTiles, rank_elem(e));
      rank_add(s.buf[1] + sg.elem_off, s.rank + sg.elem_off + q, groups, q0, lo, e);
    }
  }
}

int sort_seg_tiles(int n) { return (n + kTileR - 1) / kTileR; }
int sort_seg_items(int n) {
  const int tiles = sort_seg_tiles(n);
  return tiles > 1 ? tiles * ((tiles + kRankTiles - 1) / kRankTiles) : 0;
}

hipError_t launch_seg_sort(hipStream_t st, const SortArgs& s, const SegSort& g) {
  // twice what is resident at once (32 KB and 68 KB of LDS), in strides past it
  const int cap = 2048;
  hipLaunchKernelGGL(k_seg_tile_sort, dim3(g.tiles < cap ? g.tiles : cap), dim3(kTSBlk), 0, st,
                     s, g);
  if (g.items > 0)
    hipLaunchKernelGGL(k_seg_merge, dim3(g.items < cap ? g.items : cap), dim3(kRankBlk), 0, st,
                       s, g);
  return hipGetLastError();
}

// ------------------------------------------------------------ merge passes

// Merge-path splits of one output tile: the number of A elements among the
// first d0 (threads 0..127) and d1 (threads 128..255) outputs of merge(A, B),
// i.e. the first i with A[i] > B[d-1-i] (or the upper end of the range).
// Found by a cooperative 128-ary search: each round every thread tests one
// position, which shrinks the range by a factor of 128; the tests are
// monotone in the position, so the first true one is the count of false
// ones, summed from the two wave ballots of the half.  Every thread of the
// workgroup must call it; the splits of both halves land in s_res[0..1].
__device__ void merge_splits(const SortElem* A, int la, const SortElem* B, int lb, int d0, int d1,
                             int* s_cnt /* 4 */, int* s_done /* 2 */, int* s_res /* 2 */) {
  const int half = threadIdx.x >> 7;
  const int t = threadIdx.x & 127;
  const int wave = threadIdx.x >> 6;
  const int d = half ? d1 : d0;
  int lo = d - lb > 0 ? d - lb : 0;
  int hi = d < la ? d : la;
  for (int it = 0; it < 8; it++) {  // 128^5 > 2^31: the loop always converges before 8
    if (t == 0) s_done[half] = lo == hi;
    __syncthreads();
    const bool done = s_done[0] && s_done[1];
    if (done) break;
    const int span = hi - lo;
    int step = (span + 127) / 128;
    if (step < 1) step = 1;
    const int pos = lo + t * step;
    bool test = true;
    if (span > 0 && pos < hi) test = elem_lt(B[d - 1 - pos], A[pos]);
    const unsigned long long falses = __ballot(!test);
    if ((threadIdx.x & 63) == 0) s_cnt[wave] = __popcll(falses);
    __syncthreads();
    if (span > 0) {
      // positions lo + u*step are false for u < first and true at u = first
      const int first = s_cnt[2 * half] + s_cnt[2 * half + 1];
      int nlo = first == 0 ? lo : lo + (first - 1) * step + 1;
      const int cap = lo + first * step;
      const int nhi = cap < hi ? cap : hi;
      if (nlo > nhi) nlo = nhi;
      lo = nlo;
      hi = nhi;
    }
  }
  if (t == 0) s_res[half] = lo;
  __syncthreads();
}

// Element i of the run of length len staged at sm[r0..], or the largest
// element past its end; the index is clamped into the staging tile so the
// load is always an in-bounds LDS load.
__device__ __forceinline__ SortElem staged_head(const SortElem* sm, int r0, int i, int len) {
  int li = r0 + (i < len ? i : len - 1);
  li = li < 0 ? 0 : (li < kTileS ? li : kTileS - 1);
  return elem_sel(i < len, sm[li], kMaxElem);
}

__global__ __launch_bounds__(kSortBlk) void k_merge_pass(SortArgs s, int L, int from) {
  const int N = *s.count;
  if (!sort_enabled(s)) return;
  if (L >= N) return;
  const SortElem* src = s.buf[from];
  SortElem* dst = s.buf[from ^ 1];
  __shared__ SortElem sm[kTileS];
  __shared__ int s_cnt[4], s_done[2], s_res[2];
  const int ntiles = (N + kTileS - 1) / kTileS;
  for (int tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
    const long long o0 = (long long)tile * kTileS;
    const long long o1 = o0 + kTileS < N ? o0 + kTileS : N;
    const long long pb = (o0 / (2ll * L)) * (2ll * L);
    const int la = (int)(pb + L < N ? L : N - pb);
    const int lb = (int)(pb + 2ll * L < N ? L : (N - pb - la > 0 ? N - pb - la : 0));
    const SortElem* A = src + pb;
    const SortElem* B = src + pb + la;
    const int d0 = (int)(o0 - pb), d1 = (int)(o1 - pb);
    merge_splits(A, la, B, lb, d0, d1, s_cnt, s_done, s_res);
    const int a0 = s_res[0], a1 = s_res[1];
    const int b0 = d0 - a0, b1 = d1 - a1;
    const int na = a1 - a0, nb = b1 - b0;
    for (int j = threadIdx.x; j < na + nb; j += kSortBlk)
      sm[j] = j < na ? A[a0 + j] : B[b0 + (j - na)];
    __syncthreads();
    // each thread merges kPerThr consecutive outputs of the tile
    const int d = threadIdx.x * kPerThr;
    if (d < na + nb) {
      int lo = d - nb > 0 ? d - nb : 0;
      int hi = d < na ? d : na;
      while (lo < hi) {
        int mid = (lo + hi) >> 1;
        if (elem_lt(sm[na + (d - 1 - mid)], sm[mid])) hi = mid; else lo = mid + 1;
      }
      int ia = lo, ib = d - lo;
      // run heads in registers, an exhausted run showing the largest
      // element (no element of a sort equals it)
      SortElem ha = staged_head(sm, 0, ia, na);
      SortElem hb = staged_head(sm, na, ib, nb);
      for (int k = 0; k < kPerThr && d + k < na + nb; k++) {
        const bool ta = !elem_lt(hb, ha);
        dst[o0 + d + k] = elem_sel(ta, ha, hb);
        ia += ta;
        ib += !ta;
        const SortElem nx = staged_head(sm, ta ? 0 : na, ta ? ia : ib, ta ? na : nb);
        ha = elem_sel(ta, nx, ha);
        hb = elem_sel(ta, hb, nx);
      }
    }
    __syncthreads();
  }
}

hipError_t launch_sort(hipStream_t st, const SortArgs& s, int64_t max_count, int grid) {
  if (s.rank != nullptr && max_count <= kRankMaxCount) {
    rank_sort(st, s, max_count);
    return hipGetLastError();
  }
  const int bs_grid = s.side_ids != nullptr && grid < kSideGrid ? kSideGrid : grid;
  hipLaunchKernelGGL(k_block_sort, dim3(bs_grid), dim3(kBSBlk), 0, st, s);
  int from = 0;
  for (int64_t L = kTileB; L < max_count; L <<= 1, from ^= 1)
    hipLaunchKernelGGL(k_merge_pass, dim3(grid), dim3(kSortBlk), 0, st, s, (int)L, from);
  return hipGetLastError();
}

}  // namespace plc
