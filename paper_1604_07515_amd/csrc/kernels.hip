// kernels.hip -- gfx950 kernels of the plain (one query at a time) path:
// round-synchronous PR-Nibble (Sec. 3.3) and the parallel sweep cut
// (Sec. 3.1, Theorem 1).
//
// Round t of PR-Nibble is three launches:
//   k_self    vertexMap(Frontier, UpdateSelf): snapshot rho_v = r[v], update
//             p[v] and r[v], compute the per-entry coefficient cn*rho/d(v), and
//             (single-pass decoupled look-back scan) the start of each entry's
//             edges in the round's flattened edge sequence; entries record the
//             entry index of every 1024-edge tile they start.
//   k_scatter edgeMap(G, Frontier, UpdateNgh): one workgroup per edge tile
//             (persistent grid), entries staged in LDS, coalesced neighbour
//             reads, FP64 atomic add into r[w].  The filter of the paper is
//             folded in: r only grows during a scatter, so w joins the next
//             frontier exactly when one atomic's (old, old + c) pair straddles
//             eps*d(w); that atomic appends w.  On rounds of at least the
//             binning threshold it is pass A of the binned scatter instead
//             (pairs sorted into destination bins).
//   k_bin_apply  pass B of a binned round (LDS sums per bin, one update per
//             touched destination); it exits at once on the other rounds.
//             The host leaves it out where no round can bin, and in a
//             query's first chunk behind the launches where recent queries
//             had no round large enough (k_scatter then takes the atomic
//             form whatever the round's size).
// Rounds that cover a good part of the arcs are dense: one launch of k_dense
// each, queued in a row once a query has got there.
// A frontier of at most one scan block is handled by k_self alone: its
// workgroup 0 runs such rounds back to back (self step, scan, edge
// scatter, round close) until the frontier grows, empties or a round has
// too many edges for one workgroup; k_scatter then pushes only rounds whose
// entries were built in memory.
// Kernels read the round number and frontier size from the device control
// block and return at once when the query has finished, so rounds (and the
// sweep, guarded the same way) can be queued ahead of the host's
// termination check.
//
// The sweep: k_sweep_keys, the sort (sort.hip; its first launch also
// gathers the nonzeros of r over the touched list and resets r, on the
// workgroups that hold no tile), k_vol_scan, k_cut_count and k_cut_scan (which
// also resets p and the ranks, and takes the best prefix).
//
// Arithmetic matches the paper's updates evaluated in a fixed way: the
// constants cs, cn, keep are rounded once, p[v] + cs*rho, keep*rho and
// (cn*rho)/d are each rounded separately (the library is built with
// -ffp-contract=off), and the threshold is eps*(double)d.  Only the order of
// the atomic additions into r differs from a sequential evaluation.
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "device_util.h"
#include "plc_device.h"
#include "sort.h"

namespace plc {

// ---------------------------------------------------------------- init

__global__ void k_graph_init(PlainArgs a) {
  for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < a.n;
       v += (int64_t)gridDim.x * blockDim.x) {
    VRec rec;
    rec.r = 0.0;
    rec.deg = (int32_t)(a.off[v + 1] - a.off[v]);
    rec.rank = 0;
    a.vr[v] = rec;
    a.p[v] = 0.0;
    a.hk_r1[v] = 0.0;
    if (a.cd[0]) {
      a.cd[0][v] = 0.0;
      a.cd[1][v] = 0.0;
    }
  }
}

__device__ __forceinline__ void reset_round_book(Ctl* c) {
  c->init_held = 0;
  c->pend = 0;
  c->selfed = -1;
  c->steps = 0;
  c->loop_rounds = 0;
  c->loop_pushes = 0;
  c->loop_edges = 0;
  c->bin_rounds = 0;
  c->bin_pairs = 0u;
  c->pull_rounds = 0;
  c->bin_edges = 0;
  c->t_start = (long long)wall_clock64();
  c->t_end = 0;
  c->dense = DN_LIST;
  c->enext = 0;
  c->fill = 0;
  c->pairs0 = 0;
  c->dsteps = 0;
  c->dself = 0;
}

// Seed initialisation (Fig. alg:pr-nibble: r = {(x,1)}, Frontier = {x}).
__device__ void query_init_body(const PlainArgs& a, int32_t seed, int32_t rule, double alpha,
                                double eps, int32_t max_rounds, double beta) {
  Ctl* c = a.ctl;
  if (rule == 1) {  // original rule
    c->cs = alpha;
    c->cn = (1.0 - alpha) / 2.0;
    c->keep = (1.0 - alpha) / 2.0;
    c->opt_rule = 0;
  } else {          // optimized rule
    c->cs = 2.0 * alpha / (1.0 + alpha);
    c->cn = (1.0 - alpha) / (1.0 + alpha);
    c->keep = 0.0;
    c->opt_rule = 1;
  }
  c->eps = eps;
  c->seed = seed;
  c->rule = rule;
  c->max_rounds = max_rounds;
  c->beta = beta;
  c->beta_nf = 0;
  c->beta_k = 0;
  c->round = 0;
  c->cnt[0] = 1;
  c->cnt[1] = 0;
  c->ntiles = 0;
  c->etotal = 0;
  c->pushes = 0;
  c->edges = 0;
  c->support_cnt = 0;
  c->touched_cnt = 1;
  c->fault = 0;
  c->limited = 0;
  c->N = 0;
  c->sort_flip = 0;
  c->rnnz = 0;
  c->vol_total = a.vol_total;
  c->best_cut = 0;
  c->best_vol = 0;
  c->best_den = 0;
  c->kstar = 0;
  c->phi = 0.0;
  reset_round_book(c);
  a.fbuf0[0] = seed;
  a.touched[0] = seed;
  a.vr[seed].r = 1.0;
  c->status = ST_PUSH;
}

__global__ void k_query_init(PlainArgs a, int32_t seed, int32_t rule, double alpha, double eps,
                             int32_t max_rounds, double beta) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  query_init_body(a, seed, rule, alpha, eps, max_rounds, beta);
}

// The same, only after a swept query (or none since the graph was loaded);
// otherwise the previous query's state is left as it is.
__global__ void k_query_init_guarded(PlainArgs a, int32_t seed, int32_t rule, double alpha,
                                     double eps, int32_t max_rounds) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  Ctl* c = a.ctl;
  if (c->status != ST_SWEPT && c->status != ST_IDLE) {
    c->init_held = 1;
    return;
  }
  query_init_body(a, seed, rule, alpha, eps, max_rounds, 1.0);
}

// Seed-set initialisation (Sec. 3: a set S of seeds): the host has placed
// the distinct seeds in the first frontier; each gets r = 1/|S| and is
// listed as touched.  Block 0 also sets up the control block.
__global__ void k_query_init_set(PlainArgs a, int32_t nseeds, int32_t rule, double alpha,
                                 double eps, int32_t max_rounds) {
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    Ctl* c = a.ctl;
    if (rule == 1) {  // original rule
      c->cs = alpha;
      c->cn = (1.0 - alpha) / 2.0;
      c->keep = (1.0 - alpha) / 2.0;
      c->opt_rule = 0;
    } else {          // optimized rule
      c->cs = 2.0 * alpha / (1.0 + alpha);
      c->cn = (1.0 - alpha) / (1.0 + alpha);
      c->keep = 0.0;
      c->opt_rule = 1;
    }
    c->eps = eps;
    c->seed = a.fbuf0[0];
    c->rule = rule;
    c->max_rounds = max_rounds;
    c->beta = 1.0;
    c->beta_nf = 0;
    c->beta_k = 0;
    c->round = 0;
    c->cnt[0] = nseeds;
    c->cnt[1] = 0;
    c->ntiles = 0;
    c->etotal = 0;
    c->pushes = 0;
    c->edges = 0;
    c->support_cnt = 0;
    c->touched_cnt = nseeds;
    c->fault = 0;
    c->limited = 0;
    c->N = 0;
    c->sort_flip = 0;
    c->rnnz = 0;
    c->vol_total = a.vol_total;
    c->best_cut = 0;
    c->best_vol = 0;
    c->best_den = 0;
    c->kstar = 0;
    c->phi = 0.0;
    reset_round_book(c);
    c->status = ST_PUSH;
  }
  const double share = 1.0 / (double)nseeds;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < nseeds; i += gridDim.x * blockDim.x) {
    const int32_t v = a.fbuf0[i];
    a.touched[i] = v;
    a.vr[v].r = share;
  }
}

// ---------------------------------------------------------------- round

// The head of the control block, read at once: without the pin the compiler
// loads each field behind the test of the one before, a chain of cache
// misses at the start of every launch.
struct CtlHead {
  int32_t status, round, cnt0, cnt1, dense, selfed, max_rounds;
  double beta;
  __device__ int nf() const { return (round & 1) ? cnt1 : cnt0; }
};
__device__ __forceinline__ CtlHead ctl_head(const Ctl* c) {
  CtlHead h{c->status, c->round, c->cnt[0], c->cnt[1], c->dense, c->selfed, c->max_rounds,
            c->beta};
  asm volatile("" : "+s"(h.status), "+s"(h.round), "+s"(h.cnt0), "+s"(h.cnt1), "+s"(h.dense),
               "+s"(h.selfed), "+s"(h.max_rounds), "+s"(h.beta));
  return h;
}
// The same with what else of that line the scatter takes.
struct CtlEdges {
  int32_t ntiles;
  long long etotal;
  double eps;
};
__device__ __forceinline__ CtlHead ctl_head(const Ctl* c, CtlEdges* edges) {
  CtlEdges q{c->ntiles, c->etotal, c->eps};
  const CtlHead h = ctl_head(c);
  asm volatile("" : "+s"(q.ntiles), "+s"(q.etotal), "+s"(q.eps));
  *edges = q;
  return h;
}

__device__ __forceinline__ bool push_active(const CtlHead& h, int64_t ncap, int* t_out,
                                            int* nf_out) {
  int nf = h.nf();
  if (h.status != ST_PUSH || nf <= 0) return false;
  if ((int64_t)nf > ncap) nf = (int)ncap;
  *t_out = h.round;
  *nf_out = nf;
  return true;
}

// Entry i covers edges [s, s + d) of the round; record it as the first entry
// of every tile that starts inside that range.
__device__ __forceinline__ void mark_tiles(int32_t* tile_start, int64_t cap, long long s,
                                           long long d, int i, int* fault) {
  long long t0 = (s + kEdgeTile - 1) / kEdgeTile;
  long long t1 = (s + d - 1) / kEdgeTile;
  if (t1 >= cap) { *fault = 1; t1 = cap - 1; }
  for (long long tt = t0; tt <= t1; tt++) tile_start[tt] = i;
}

// Round rules sharing the round kernels.
enum : int { kModePR = 0, kModeHK = 1, kModeNB = 2 };

// HK-PR residual (Nibble vector) of vertex v at level (iteration) k: even
// levels in the state record, odd levels in hk_r1.
__device__ __forceinline__ double* hk_res(const PlainArgs& a, int k, int32_t v) {
  return (k & 1) ? &a.hk_r1[v] : &a.vr[v].r;
}

// vertexMap(Frontier, UpdateSelf) + degree scan of the frontier.
//   PR-Nibble (Figs. alg:pr-nibble / alg:pr-nibble2): p += cs rho, r =
//     keep rho (-0.0 under the optimized rule), coefficient cn rho / d.
//   HK-PR level j (Fig. alg:hkpr): p += rho; coefficient t rho / ((j+1) d),
//     or rho / d on the last level; first, the residuals of level j - 1
//     (the array level j + 1 fills) are cleared over the vertices that
//     level touched.
//   Nibble step j -> j+1 (Fig. alg:nibble): coefficient rho / (2 d), and
//     rho / 2 kept per entry for the scatter, which adds it to the vertex's
//     own next value; the same clearing as HK-PR.
//   LIGHT (a round handed back by the dense form): the self step was taken
//     there; the entries take their coefficients from cd[t & 1], which is
//     cleared again.
template <int MODE, bool LIGHT, int NT>
__device__ __forceinline__ void self_body(const PlainArgs& a, int slot, const CtlHead& h) {
  constexpr bool HK = MODE == kModeHK;
  constexpr int kItems = kScanBlock / NT;  // entries per thread
  constexpr bool LEVELS = MODE != kModePR;
  Ctl* c = a.ctl;
  int t, nf;
  if (!push_active(h, a.n, &t, &nf)) return;
  if (LEVELS) {
    if (t >= (HK ? c->hk_N : h.max_rounds)) return;  // (the host queues no more)
    if (t >= 1) {
      const int lp = (t + 2) % 3;
      const int np = c->hk_tlc[lp];
      const int32_t* Lp = a.hk_tl[lp];
      for (int i = blockIdx.x * NT + threadIdx.x; i < np; i += gridDim.x * NT)
        *hk_res(a, t + 1, Lp[i]) = 0.0;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) c->hk_tlc[(t + 1) % 3] = 0;
  } else if (t >= h.max_rounds) {
    if (blockIdx.x == 0 && threadIdx.x == 0) { c->limited = 1; c->status = ST_LIMIT; }
    return;
  }
  __shared__ long long sh[NT / 64 + 1];
  __shared__ long long s_excl;
  __shared__ unsigned long long s_tk;
  __shared__ int32_t s_sup[kScanBlock];
  __shared__ int32_t s_stay[LEVELS ? 1 : kScanBlock];
  __shared__ int s_nsup, s_nstay, s_base;
  const int nblk = (nf + kScanBlock - 1) / kScanBlock;
  const bool fixed = !LIGHT && scan_fixed(nblk);
  if (fixed && (int)blockIdx.x >= nblk) return;
  ScanSite* site = &c->scan[SCAN_FRONTIER];
  unsigned long long* desc;
  const int32_t* F = (t & 1) ? a.fbuf1 : a.fbuf0;
  int32_t* Fn = (t & 1) ? a.fbuf0 : a.fbuf1;
  int32_t* cntn = &c->cnt[(t + 1) & 1];
  const double cs = c->cs, cn = c->cn, keep = c->keep, eps = c->eps;
  const bool opt = LEVELS || c->opt_rule != 0;
  const bool hk_last = HK && t + 1 == c->hk_N;
  const double hk_t = HK ? c->hk_t : 0.0;
  double* const cd = LIGHT ? a.cd[t & 1] : nullptr;
  if (threadIdx.x == 0) { s_nsup = 0; s_nstay = 0; }
  for (int b = scan_begin(site, a.desc[SCAN_FRONTIER], a.desc_cap, nblk, fixed, &s_tk, &desc);
       b < nblk; b = scan_next(site, nblk, fixed, &s_tk)) {
    // each thread takes kItems consecutive entries: one workgroup scan
    // of the per-thread sums, then a serial prefix inside the thread.  All
    // loads of the thread's entries go out together, before any store (entry
    // by entry they were a chain of 6 us for a block, 2 us so).
    const int i0 = b * kScanBlock + (int)threadIdx.x * kItems;
    int32_t dk[kItems], vk[kItems];
    const int mine = nf - i0;  // entries of this thread (may be < 0, or more than it takes)
    if (mine >= kItems) {
      if constexpr (kItems == 4) {
        const int4 f = *reinterpret_cast<const int4*>(F + i0);
        vk[0] = f.x; vk[1] = f.y; vk[2] = f.z; vk[3] = f.w;
      } else {
#pragma unroll
        for (int k = 0; k < kItems; k++) vk[k] = F[i0 + k];
      }
    } else {
#pragma unroll
      for (int k = 0; k < kItems; k++) vk[k] = F[k < mine ? i0 + k : 0];
    }
    VRec rec[kItems];
    double xk[kItems], pk[kItems];
    int64_t rk[kItems];
#pragma unroll
    for (int k = 0; k < kItems; k++) {
      const int32_t v = vk[k];
      rec[k] = a.vr[v];
      xk[k] = LIGHT ? cd[v] : LEVELS && (t & 1) ? a.hk_r1[v] : rec[k].r;
      pk[k] = MODE == kModeNB || LIGHT ? 1.0 : a.p[v];
      rk[k] = a.off[v];
    }
    long long dsum = 0;
    unsigned sup = 0, stay = 0;  // bit k: entry k
#pragma unroll
    for (int k = 0; k < kItems; k++) {
      const int i = i0 + k;
      const int32_t v = vk[k];
      dk[k] = 0;
      if (k >= mine) continue;
      const int32_t d = rec[k].deg;
      const double rho = xk[k];
      dk[k] = d;
      dsum += d;
      if (pk[k] == 0.0) sup |= 1u << k;
      if (LIGHT) {
        a.coef[i] = rho;  // (the coefficient itself)
        cd[v] = 0.0;
        if (!opt && rec[k].r >= eps * (double)d) stay |= 1u << k;  // (r is keep rho already)
      } else if (MODE == kModeNB) {
        a.coef[i] = rho / (2.0 * (double)d);
        a.sp[i] = rho / 2.0;
      } else if (HK) {
        a.p[v] = pk[k] + rho;
        a.coef[i] = hk_last ? rho / (double)d : (hk_t * rho) / ((double)(t + 1) * (double)d);
      } else {
        a.p[v] = pk[k] + cs * rho;
        const double nr = opt ? -0.0 : keep * rho;
        a.vr[v].r = nr;
        a.coef[i] = (cn * rho) / (double)d;
        if (!opt && nr >= eps * (double)d) stay |= 1u << k;
      }
      a.rowp[i] = rk[k];
    }
    if (!opt) wave_append_all<kItems>(stay, vk, s_stay, &s_nstay);
    if (MODE != kModeNB && !LIGHT) wave_append_all<kItems>(sup, vk, s_sup, &s_nsup);
    long long agg;
    const long long ex = block_excl_scan<NT>(dsum, &agg, sh);
    if (threadIdx.x < 64) {
      const long long ex0 = scan_lookback(desc, b, agg, &c->fault);
      if (threadIdx.x == 0) s_excl = ex0;
    }
    __syncthreads();
    long long s = s_excl + ex;
#pragma unroll
    for (int k = 0; k < kItems; k++) {
      const int i = i0 + k;
      if (i < nf) {
        a.estart[i] = s;
        mark_tiles(a.tile_start, a.tile_cap, s, dk[k], i, &c->fault);
      }
      s += dk[k];
    }
    if (b == nblk - 1 && threadIdx.x == 0) {
      const long long tot = s_excl + agg;
      c->etotal = tot;
      c->ntiles = (int)((tot + kEdgeTile - 1) / kEdgeTile);
      c->selfed = t;
      c->steps += 1;
      if (slot >= 0) a.work_log[2 * slot] = 1;
    }
    if (MODE != kModeNB && !LIGHT)
      block_flush(&c->support_cnt, a.support, a.n, s_sup, &s_nsup, &s_base, &c->fault);
    if (!opt) block_flush(cntn, Fn, a.n, s_stay, &s_nstay, &s_base, &c->fault);
  }
  // (every workgroup has read the state it decided on by the time the last
  // one gets here)
  if (LIGHT && last_block(&c->done[DONE_DENSE], &s_base, false) && threadIdx.x == 0) {
    c->dense = DN_LIST;
    c->cd_dirty = 0;
  }
}

// Whether the addition of c that returned `old` is the first touch of a word
// that was +0.0.  A c that underflowed to 0 (HK-PR and Nibble, whose eps may be
// any positive number) leaves the word as it was and touches nothing: counted,
// every such addition would be a first one, more of them than the lists hold.
__device__ __forceinline__ bool first_touch(double old, double c) {
  return __double_as_longlong(old) == 0 && c != 0.0;
}

// Threshold decision for one addition of c to r[w] that returned `old`
// (lanes without an addition pass valid = false): crossing appends w to the
// next frontier, first touch to the touched list (wave-ballot appends).
__device__ __forceinline__ void decide(bool valid, double old, double c, double thr, int32_t w,
                                       int32_t* s_fn, int* s_nfn, int32_t* s_tv, int* s_ntv) {
  wave_append(valid && old < thr && old + c >= thr, w, s_fn, s_nfn);
  wave_append(valid && first_touch(old, c), w, s_tv, s_ntv);
}

template <typename T>
__device__ __forceinline__ T ld_agent(T* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ __forceinline__ void st_agent(T* p, T v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Append the n values of buf at dst[base..] (capacity cap) and, where
// mirror is set, at mirror[base..] below kScanBlock.  The caller's
// workgroup is the only writer of the list, so the base is its own count.
__device__ __forceinline__ void local_append(int32_t* dst, int64_t cap, int32_t* mirror,
                                             const int32_t* buf, int n, int base, int* fault) {
  for (int j = threadIdx.x; j < n; j += kSelfBlk) {
    const long long slot = (long long)base + j;
    if (slot < cap) dst[slot] = buf[j]; else *fault = 1;
    if (mirror && slot < kScanBlock) mirror[slot] = buf[j];
  }
}

// Rounds with small frontiers (Figs. alg:pr-nibble / alg:pr-nibble2, the
// same updates and arithmetic as k_self + k_scatter), run back to back by
// workgroup 0 alone: the frontier (at most kScanBlock vertices) and its
// entries stay in LDS, list lengths are kept locally, and only the FP64
// additions into r go to memory as device-scope atomics.  r of the frontier
// is read and written with device-scope atomic accesses too, so that within
// the launch they are ordered with those additions.  It stops when the
// frontier empties or outgrows a scan block, when a round has more than
// kLoopEdges edges (that round's entries are then built in memory for the
// next scatter launch, exactly as k_self builds them), at the round limit, or
// after kLoopMaxRounds rounds.
__device__ void loop_rounds(const PlainArgs& a, int slot, int t, int nf) {
  Ctl* c = a.ctl;
  constexpr int kItems = kScanBlock / kSelfBlk;  // entries per thread
  __shared__ int32_t s_F[2][kScanBlock];  // this round's and the next round's frontier
  __shared__ int32_t s_est[kScanBlock];   // entry i: first edge in the round's edge sequence
  __shared__ int64_t s_row[kScanBlock];   //          off[v]
  __shared__ double s_cf[kScanBlock];     //          cn rho / d(v)
  __shared__ unsigned short s_own[kLoopPass];  // edge of the pass: its entry's place
  __shared__ int32_t s_fn[kLoopPass];     // crossings of one pass
  __shared__ int32_t s_tv[kLoopPass];     // first touches of one pass
  __shared__ int32_t s_sup[kScanBlock];
  __shared__ int32_t s_stay[kScanBlock];
  __shared__ long long sh[kSelfBlk / 64 + 1];
  __shared__ int s_nfn, s_ntv, s_nsup, s_nstay;
  if (threadIdx.x == 0) {
    s_nfn = 0;
    s_ntv = 0;
    s_nsup = 0;
    s_nstay = 0;
  }
  __syncthreads();
  const double cs = c->cs, cn = c->cn, keep = c->keep, eps = c->eps;
  const bool opt = c->opt_rule != 0;
  const int max_rounds = c->max_rounds;
  const int64_t cap = a.n;
  int tcnt = c->touched_cnt, scnt = c->support_cnt;
  long long pushes = 0, edges = 0, E = 0;
  int nnext = 0, cur = 0, rounds = 0;
  bool selfed = false;
  for (int it = 0;; it++) {
    const int32_t* F = it > 0 ? s_F[cur] : (t & 1) ? a.fbuf1 : a.fbuf0;
    int32_t* Fn = (t & 1) ? a.fbuf0 : a.fbuf1;
    // vertexMap(Frontier, UpdateSelf) and the degree scan.  Thread j's entries
    // are the frontier's j, j + kSelfBlk, ... (a small frontier is one entry per
    // thread), kept at places per j, per j + 1, ...: a place past the frontier
    // holds an entry of no edges.  All loads go out before any store.
    const int per = (nf + kSelfBlk - 1) / kSelfBlk;
    int32_t dk[kItems], vk[kItems];
    double ck[kItems], xk[kItems], pk[kItems];
    int64_t rk[kItems];
    const int mine = (nf - (int)threadIdx.x + kSelfBlk - 1) / kSelfBlk;  // (may be < 0)
#pragma unroll
    for (int k = 0; k < kItems; k++) vk[k] = k < mine ? F[k * kSelfBlk + (int)threadIdx.x] : 0;
#pragma unroll
    for (int k = 0; k < kItems; k++) {
      dk[k] = 0;
      xk[k] = 0.0;
      pk[k] = 0.0;
      rk[k] = 0;
      if (k < mine) {
        dk[k] = a.vr[vk[k]].deg;
        xk[k] = ld_agent(&a.vr[vk[k]].r);
        pk[k] = a.p[vk[k]];
        rk[k] = a.off[vk[k]];
      }
    }
    long long dsum = 0;
    unsigned sup = 0, stay = 0;  // bit k: entry k
#pragma unroll
    for (int k = 0; k < kItems; k++) {
      ck[k] = 0.0;
      if (k >= mine) continue;
      const double rho = xk[k];
      const double nr = opt ? -0.0 : keep * rho;
      dsum += dk[k];
      ck[k] = (cn * rho) / (double)dk[k];
      if (!opt && nr >= eps * (double)dk[k]) stay |= 1u << k;
      if (pk[k] == 0.0) sup |= 1u << k;
      a.p[vk[k]] = pk[k] + cs * rho;
      st_agent(&a.vr[vk[k]].r, nr);
    }
    if (!opt) wave_append_all<kItems>(stay, vk, s_stay, &s_nstay);
    wave_append_all<kItems>(sup, vk, s_sup, &s_nsup);
    long long agg;
    const long long ex = block_excl_scan<kSelfBlk>(dsum, &agg, sh);
    E = agg;
    const int nstay = s_nstay, nsup = s_nsup;
    local_append(a.support, cap, nullptr, s_sup, nsup, scnt, &c->fault);
    local_append(Fn, cap, s_F[cur ^ 1], s_stay, nstay, 0, &c->fault);
    scnt += nsup;
    nnext = nstay;
    if (E > kLoopEdges) {
      // too large for one workgroup: entries in memory for the scatter
      // launch, at consecutive places (those of no edges left out: the
      // threads before this one hold per entries each, or the frontier's
      // rest), and the frontier in the same order
      int32_t* const Fo = (t & 1) ? a.fbuf1 : a.fbuf0;
      long long s = ex;
      const int full = nf - (per - 1) * kSelfBlk;  // threads with per entries
      const int j = (int)threadIdx.x;
      int i = j <= full ? j * per : full * per + (j - full) * (per - 1);
#pragma unroll
      for (int k = 0; k < kItems; k++) {
        if (k < mine) {
          Fo[i] = vk[k];
          a.estart[i] = s;
          a.rowp[i] = rk[k];
          a.coef[i] = ck[k];
          mark_tiles(a.tile_start, a.tile_cap, s, dk[k], i, &c->fault);
          i++;
        }
        s += dk[k];
      }
      selfed = true;
      break;
    }
    {
      long long s = ex;
#pragma unroll
      for (int k = 0; k < kItems; k++) {
        if (k < per) {
          const int i = (int)threadIdx.x * per + k;
          s_est[i] = (int32_t)s;
          s_row[i] = rk[k];
          s_cf[i] = ck[k];
        }
        s += dk[k];
      }
    }
    __syncthreads();
    if (threadIdx.x == 0) { s_nstay = 0; s_nsup = 0; }
    // edgeMap(G, Frontier, UpdateNgh), kLoopPass edges per pass
    constexpr int kPer = kLoopPass / kSelfBlk;
    for (long long base = 0; base < E; base += kLoopPass) {
      // the entry of every edge of the pass: one search per thread for the
      // first of ept consecutive edges, the others follow from it; the edges
      // are then taken kSelfBlk apart (see the scatter)
      const int rest = (int)(E - base);
      const int len = rest < kLoopPass ? rest : kLoopPass;
      const int ept = (len + kSelfBlk - 1) / kSelfBlk;
      {
        const int r0 = (int)threadIdx.x * ept;
        int lo = 0, hi = per * kSelfBlk - 1;
        while (lo < hi) {
          const int mid = (lo + hi + 1) >> 1;
          if (s_est[mid] <= (int)base + r0) lo = mid; else hi = mid - 1;
        }
        for (int k = 0; k < ept && r0 + k < len; k++) {
          // (places of no edges are passed over)
          while (lo + 1 < per * kSelfBlk && s_est[lo + 1] <= (int)base + r0 + k) lo++;
          s_own[r0 + k] = (unsigned short)lo;
        }
      }
      __syncthreads();
      int32_t w[kPer];
      double cf[kPer];
#pragma unroll
      for (int k = 0; k < kPer; k++) {
        const int rel = k * kSelfBlk + (int)threadIdx.x;
        w[k] = -1;
        cf[k] = 0.0;
        if (rel < len) {
          const int at = s_own[rel];
          w[k] = a.nbr[s_row[at] + ((int)base + rel - s_est[at])];
          cf[k] = s_cf[at];
        }
      }
      int32_t dw[kPer];
#pragma unroll
      for (int k = 0; k < kPer; k++) dw[k] = w[k] >= 0 ? a.vr[w[k]].deg : 0;
      double old[kPer];
#pragma unroll
      for (int k = 0; k < kPer; k++) old[k] = w[k] >= 0 ? unsafeAtomicAdd(&a.vr[w[k]].r, cf[k]) : 0.0;
      unsigned cross = 0, touch = 0;  // bit k: edge k
#pragma unroll
      for (int k = 0; k < kPer; k++) {
        const double thr = eps * (double)dw[k];
        if (w[k] < 0) continue;
        if (old[k] < thr && old[k] + cf[k] >= thr) cross |= 1u << k;
        if (__double_as_longlong(old[k]) == 0) touch |= 1u << k;
      }
      wave_append_all<kPer>(cross, w, s_fn, &s_nfn);
      wave_append_all<kPer>(touch, w, s_tv, &s_ntv);
      __syncthreads();
      const int nfn = s_nfn, ntv = s_ntv;
      local_append(Fn, cap, s_F[cur ^ 1], s_fn, nfn, nnext, &c->fault);
      local_append(a.touched, cap, nullptr, s_tv, ntv, tcnt, &c->fault);
      nnext += nfn;
      tcnt += ntv;
      __syncthreads();
      if (threadIdx.x == 0) { s_nfn = 0; s_ntv = 0; }
      __syncthreads();
    }
    // the round is over (the barrier orders this round's LDS appends and
    // count resets before the next round's, also when E is 0)
    __syncthreads();
    pushes += nf;
    edges += E;
    rounds += 1;
    t += 1;
    nf = nnext;
    nnext = 0;
    cur ^= 1;
    if (nf == 0 || nf > kScanBlock || t >= max_rounds || it + 1 >= kLoopMaxRounds) break;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    c->touched_cnt = tcnt;
    c->support_cnt = scnt;
    c->pushes += pushes;
    c->edges += edges;
    c->loop_rounds += rounds;
    c->loop_pushes += pushes;
    c->loop_edges += edges;
    c->steps += 1;
    if (selfed) {
      c->etotal = E;
      c->ntiles = (int)((E + kEdgeTile - 1) / kEdgeTile);
    }
    // The launch's other workgroups may only now read these words.  They leave
    // where they see a frontier of at most a scan block, so no larger one is
    // put there: the scatter launch does that (pend).
    const bool large = !selfed && nf > kScanBlock;
    c->cnt[(t + 1) & 1] = nnext;  // stays of a round left to the scatter launch
    c->cnt[t & 1] = large ? 0 : nf;
    c->pend = large ? nf : 0;
    c->selfed = selfed ? t : -1;
    c->round = t;
    if (slot >= 0) a.work_log[2 * slot] = 1;
  }
}

// ---------------------------------------------------------------- dense rounds
//
// A round whose frontier's edges are a good part of the graph's arcs needs
// neither atomics nor pairs: every row w sums the coefficients of its
// neighbours, read from the dense array cd[t & 1] (+0.0 off the frontier).  The
// row's sum is complete in one place, so the same lane takes w's next self
// step at once (p, r, and w's coefficient for round t + 1 into
// cd[(t + 1) & 1]): a round is one launch with no frontier list.
// Bound: one random 8-byte load of cd per arc (the neighbour ids stream).
// A workgroup takes a block of rows with at most kDenseArcs arcs, so that its
// products fit 16 KB of LDS and seven workgroups share a CU; rows are then
// summed by 256 / rows lanes each, and a block's rows times its longest row
// is bounded (kDenseSpan) so that a lane sums fewer than 128 products: 256 /
// rows lanes would have 64 at most, and are a power of two.  Longer rows are cut
// into pieces that add up in dacc; the last piece finishes the row.

struct DenseLds {
  double prod[kDenseArcs];
  double sum[kDenseRows];
  int roff[kDenseRows + 1];
  int32_t sup[kDenseRows], tv[kDenseRows], fn[kDenseRows];
  double wsum[kBlock / 64];
  long long wcnt[2 * kBlock / 64];
  int nsup, ntv, nfn, base;
};

// A round of E edges is cheaper dense: a dense round costs one launch and
// every arc once, the other forms a launch more (about kDenseBase arcs'
// worth) and about kDenseRatio times as much per edge.
__device__ __forceinline__ bool dense_pays(const PlainArgs& a, long long E) {
  if (a.cd[0] == nullptr) return false;
  if (a.dense_free) return a.vol_total <= kDenseBase + kDenseRatio * E;
  return E >= a.bin_emin && E >= a.dense_emin;
}

// Whether the dense round t takes the next self step too: not if the push may
// not go on or the next frontier has to be ranked first (beta); PR-Nibble then
// lists the next frontier.
template <int MODE>
__device__ __forceinline__ bool dense_fuses(const Ctl* c, int t) {
  return MODE == kModeHK ? t + 1 < c->hk_N : t + 1 < c->max_rounds && c->beta >= 1.0;
}

// The frontier of round t as the dense round before it counted it (counts of
// an earlier launch), by one whole wave; the counts are cleared.
__device__ __forceinline__ int dense_count(const PlainArgs& a, int t) {
  static_assert(kDenseGroups == 64, "one group per lane");
  int x = a.dgrp[PLC_LANE].nf[t & 1];
  a.dgrp[PLC_LANE].nf[t & 1] = 0;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o);
  return x;
}

struct DenseCtl {
  int32_t opt_rule, cd_dirty, hk_N;
  double eps, cs, cn, keep, hk_t, hk_A;
};

// Round t in the dense form, k the workgroup's first block and b its record
// (loaded ahead of the control block).
template <int MODE>
__device__ __forceinline__ void dense_round(const PlainArgs& a, int slot, DenseLds& L, int k,
                                            DenseBlk b, const CtlHead& h,
                                            const DenseCtl& q) {
  constexpr bool HK = MODE == kModeHK;
  Ctl* c = a.ctl;
  const int t = h.round, nf = h.nf();
  const bool hk_last = HK && t + 1 == q.hk_N;
  const bool fuse = HK ? !hk_last : t + 1 < h.max_rounds && h.beta >= 1.0;
  // the list self step listed what stays, and beta carries what it did not
  // push: then only crossings join the list
  const bool listed = !fuse && h.selfed == t;
  const bool wipe = (q.cd_dirty >> ((t + 1) & 1)) & 1;
  const bool opt = q.opt_rule != 0;
  const double cs = q.cs, cn = q.cn, keep = q.keep;
  const double eps = HK ? q.hk_A : q.eps;
  const double den = HK && !hk_last ? a.hk_B[t + 1] : 1.0;
  const double hk_t = q.hk_t;
  const bool hk_next_last = HK && t + 2 == q.hk_N;
  const double* const cd = a.cd[t & 1];
  double* const cdn = a.cd[(t + 1) & 1];
  int32_t* const Fn = (t & 1) ? a.fbuf0 : a.fbuf1;
  const int tid = threadIdx.x;
  if (tid == 0) { L.nsup = 0; L.ntv = 0; L.nfn = 0; }
  long long my_nf = 0, my_e = 0;

  // the row's end: its residual, and its next self step when it is active
  auto finish = [&](bool on, int32_t w, int32_t d, double s, double rold, double pold) {
    bool sup = false, touch = false, list = false;
    on = on && d > 0;
    if (on) {
      bool act;
      double r = s;
      if (HK) {
        const double thr = (eps * (double)d) / den;
        act = !hk_last && 0.0 < thr && s >= thr;
        if (hk_last && s != 0.0) {
          a.p[w] = pold + s;
          sup = pold == 0.0;
        }
      } else {
        const double thr = eps * (double)d;
        r = rold + s;
        act = listed ? rold < thr && r >= thr : r > 0.0 && r >= thr;
        touch = s != 0.0 && __double_as_longlong(rold) == 0;
        if (!(act && fuse) && s != 0.0) a.vr[w].r = r;
      }
      double x = 0.0;
      if (act) {
        list = !fuse;
        if (fuse) {
          my_nf += 1;
          my_e += d;
          a.p[w] = HK ? pold + r : pold + cs * r;
          sup = pold == 0.0;
          if (HK) {
            x = hk_next_last ? r / (double)d : (hk_t * r) / ((double)(t + 2) * (double)d);
            // (one that underflows is kept apart from those off the frontier)
            if (x == 0.0) x = -0.0;
          } else {
            a.vr[w].r = opt ? -0.0 : keep * r;
            x = (cn * r) / (double)d;
          }
        }
      }
      if (fuse || wipe) cdn[w] = x;
    }
    wave_append(sup, w, L.sup, &L.nsup);
    if (!HK) {
      wave_append(touch, w, L.tv, &L.ntv);
      wave_append(list, w, L.fn, &L.nfn);
    }
  };

  for (;;) {
    const bool piece = b.lid >= 0;
    const int R = piece ? 1 : b.nrows;
    constexpr int kPer = kDenseArcs / kBlock;
    static_assert(kDenseRows == kBlock, "one row per thread");
    int32_t u[kPer];
#pragma unroll
    for (int j = 0; j < kPer; j++) {
      // (a block has arcs; past its last one that one is read again)
      const int e = j * kBlock + tid;
      u[j] = a.nbr[b.first + (e < b.len ? e : b.len - 1)];
    }
    // the thread's row (a piece: the row, once it is complete)
    const int32_t w = b.row + (tid < R ? tid : R - 1);
    const long long o = a.off[w];
    const VRec rec = a.vr[w];
    const double pold = a.p[w];
    double x[kPer];
#pragma unroll
    for (int j = 0; j < kPer; j++) x[j] = cd[u[j]];
    if (piece) {
      double s = 0.0;
#pragma unroll
      for (int j = 0; j < kPer; j++) s += j * kBlock + tid < b.len ? x[j] : 0.0;
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
      if (PLC_LANE == 0) L.wsum[PLC_WID] = s;
      __syncthreads();
      if (tid < 64) {  // one wave: the appends are ballots
        bool last = false;
        if (tid == 0) {
          s = 0.0;
          for (int w = 0; w < kBlock / 64; w++) s += L.wsum[w];
          // the addition has returned, so it is in place, before it is counted
          const double before = unsafeAtomicAdd(&a.dacc[b.lid], s);
          unsigned one = 1;
          asm volatile("" : "+v"(one) : "v"(before));
          last = atomicAdd(&a.dcnt[b.lid], one) == (unsigned)b.nrows - 1;
        }
        if (last) {
          s = ld_agent(&a.dacc[b.lid]);
          st_agent(&a.dacc[b.lid], 0.0);
          st_agent(&a.dcnt[b.lid], 0u);
        }
        finish(last, w, rec.deg, s, rec.r, pold);
      }
    } else {
#pragma unroll
      for (int j = 0; j < kPer; j++) L.prod[j * kBlock + tid] = x[j];
      if (tid < R) L.roff[tid] = (int)(o - b.first);
      if (tid == 0) L.roff[R] = b.len;
      __syncthreads();
      // lanes per row: a power of two, at most a wave
      int tpr = 1;
      while (2 * tpr * R <= kBlock && tpr < 64) tpr *= 2;
      const int l = tid & (tpr - 1);
      for (int i = tid / tpr; i < R; i += kBlock / tpr) {
        // (four sums: their LDS reads are in flight together)
        double s = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
        const int e1 = L.roff[i + 1];
        int e = L.roff[i] + l;
        for (; e + 3 * tpr < e1; e += 4 * tpr) {
          s += L.prod[e];
          s1 += L.prod[e + tpr];
          s2 += L.prod[e + 2 * tpr];
          s3 += L.prod[e + 3 * tpr];
        }
        for (; e < e1; e += tpr) s += L.prod[e];
        s = (s + s1) + (s2 + s3);
        for (int o = tpr >> 1; o > 0; o >>= 1) s += __shfl_xor(s, o);
        if (l == 0) L.sum[i] = s;
      }
      __syncthreads();
      finish(tid < R, w, rec.deg, tid < R ? L.sum[tid] : 0.0, rec.r, pold);
    }
    __syncthreads();
    const int nsup = L.nsup, ntv = L.ntv, nfn = L.nfn;
    if (nsup > 0) block_flush(&c->support_cnt, a.support, a.n, L.sup, &L.nsup, &L.base, &c->fault);
    if (ntv > 0) block_flush(&c->touched_cnt, a.touched, a.n, L.tv, &L.ntv, &L.base, &c->fault);
    if (nfn > 0)
      block_flush(&c->cnt[(t + 1) & 1], Fn, a.n, L.fn, &L.nfn, &L.base, &c->fault);
    k += gridDim.x;
    if (k >= a.ndblk) break;
    b = a.dblk[k];
    __syncthreads();
  }

  // the next frontier's size and edges, and the round's close.  A word that
  // all workgroups add to costs ~15 ns per addition, so groups of kDenseGroup
  // workgroups count themselves first, the edges in the same word (R-MAT 2^16,
  // 700 workgroups: 16 us per round with one word)
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    my_nf += __shfl_xor(my_nf, o);
    my_e += __shfl_xor(my_e, o);
  }
  if (PLC_LANE == 0) {
    L.wcnt[2 * PLC_WID] = my_nf;
    L.wcnt[2 * PLC_WID + 1] = my_e;
  }
  __syncthreads();
  if (tid >= 64) return;
  bool last = false;
  unsigned long long en = 0;
  if (tid == 0) {
    long long n1 = 0;
    for (int w = 0; w < kBlock / 64; w++) {
      n1 += L.wcnt[2 * w];
      en += (unsigned long long)L.wcnt[2 * w + 1];
    }
    const int G = gridDim.x, g0 = blockIdx.x / kDenseGroup * kDenseGroup;
    const int members = G - g0 < kDenseGroup ? G - g0 : kDenseGroup;
    DenseGrp* grp = &a.dgrp[blockIdx.x / kDenseGroup];
    if (n1 > 0) atomicAdd(&grp->nf[(t + 1) & 1], (int)n1);
    unsigned long long prev = atomicAdd(&grp->word, en << 16 | 1ull);
    if ((int)(prev & 0xffff) == members - 1) {
      st_agent(&grp->word, 0ull);
      en += prev >> 16;
      prev = atomicAdd(&c->enext, en << 16 | 1ull);
      last = (int)(prev & 0xffff) == (G + kDenseGroup - 1) / kDenseGroup - 1;
      en += prev >> 16;
    }
  }
  last = __shfl((int)last, 0) != 0;
  if (!last) return;
  const bool own_self = h.selfed != t;  // the self step came with the previous dense round
  const int counted = dense_count(a, t);
  if (tid != 0) return;
  const long long E = c->etotal;
  if (own_self) {
    c->steps += 1;
    c->dself += 1;
  }
  if (slot >= 0) {
    if (own_self) a.work_log[2 * slot] = 1;
    a.work_log[2 * slot + 1] = 1;
  }
  c->pushes += own_self ? counted : nf;
  c->edges += E;
  if (E >= a.bin_emin) {  // (the counters tell rounds of the binning threshold)
    c->bin_rounds += 1;
    c->pull_rounds += E >= a.dense_emin;
    c->bin_edges += E;
  }
  c->cnt[t & 1] = 0;
  if (fuse) c->cnt[(t + 1) & 1] = en > 0;
  c->etotal = (long long)en;
  c->enext = 0;
  c->dsteps += 1;
  const bool go = fuse && en > 0;
  c->dense = !go ? DN_LIST : dense_pays(a, (long long)en) ? DN_READY : DN_CONVERT;
  c->cd_dirty = (1 << (t & 1)) | (go ? 1 << ((t + 1) & 1) : 0);
  c->round = t + 1;
}

// Back to the list form: the frontier is listed from the coefficients (a 0 on
// it is -0.0, PR-Nibble has none: eps >= 1e-250 bounds its r from below), and
// the other array is cleared.
__device__ void dense_convert(const PlainArgs& a, DenseLds& L) {
  Ctl* c = a.ctl;
  const int t = c->round;
  const double* const cd = a.cd[t & 1];
  double* const old = a.cd[(t + 1) & 1];
  int32_t* const F = (t & 1) ? a.fbuf1 : a.fbuf0;
  if (threadIdx.x == 0) L.nfn = 0;
  __syncthreads();
  for (int64_t i0 = (int64_t)blockIdx.x * kBlock; i0 < a.n; i0 += (int64_t)gridDim.x * kBlock) {
    const int64_t i = i0 + threadIdx.x;
    bool in = false;
    if (i < a.n) {
      in = __double_as_longlong(cd[i]) != 0;
      old[i] = 0.0;
    }
    wave_append(in, (int32_t)i, L.fn, &L.nfn);
    block_flush(&c->fill, F, a.n, L.fn, &L.nfn, &L.base, &c->fault);
  }
  if (last_block(&c->done[DONE_DENSE], &L.base, false) && threadIdx.x < 64) {
    const int nf = dense_count(a, t);
    if (threadIdx.x != 0) return;
    if (atomicAdd(&c->fill, 0) != nf) c->fault = 1;
    c->cnt[t & 1] = nf;
    c->fill = 0;
    c->dsteps += 1;
    c->dense = DN_LIGHT;
    c->cd_dirty = 1 << (t & 1);
  }
}

template <int MODE>
__device__ __forceinline__ void dense_body(const PlainArgs& a, int slot) {
  __shared__ DenseLds L;
  const Ctl* c = a.ctl;
  const int k = blockIdx.x;  // (the grid has at most one workgroup per block)
  // the block and all of the control block that a round needs, at once
  DenseBlk b = a.dblk[k];
  DenseCtl q{c->opt_rule, c->cd_dirty, c->hk_N, c->eps,
             c->cs, c->cn, c->keep, c->hk_t, c->hk_A};
  const CtlHead h = ctl_head(c);
  asm volatile("" : "+s"(b.row), "+s"(b.nrows), "+s"(b.lid), "+s"(b.len), "+s"(b.first));
  asm volatile("" : "+s"(q.opt_rule), "+s"(q.cd_dirty), "+s"(q.hk_N),
               "+s"(q.eps), "+s"(q.cs), "+s"(q.cn), "+s"(q.keep), "+s"(q.hk_t),
               "+s"(q.hk_A));
  if (h.status != ST_PUSH || h.nf() <= 0) return;
  if (h.dense == DN_READY)
    dense_round<MODE>(a, slot, L, k, b, h, q);
  else if (h.dense == DN_CONVERT)
    dense_convert(a, L);
}
__global__ __launch_bounds__(kBlock) void k_dense(PlainArgs a, int slot) {
  dense_body<kModePR>(a, slot);
}
__global__ __launch_bounds__(kBlock) void k_hk_dense(PlainArgs a) { dense_body<kModeHK>(a, -1); }

// Entry into the dense form: the frontier's coefficients into cd[t & 1]
// (all 0 before); the next launch runs the round.  HK-PR: the level's
// residuals, which the self step has read, are cleared here (the dense form
// keeps none).
template <int MODE>
__device__ void dense_enter(const PlainArgs& a, int t, int nf, int* s_last) {
  Ctl* c = a.ctl;
  const int32_t* F = (t & 1) ? a.fbuf1 : a.fbuf0;
  double* const cd = a.cd[t & 1];
  for (int i = blockIdx.x * kBlock + threadIdx.x; i < nf; i += gridDim.x * kBlock)
    cd[F[i]] = a.coef[i];
  if (MODE == kModeHK) {
    const int np = c->hk_tlc[t % 3];
    const int32_t* Lp = a.hk_tl[t % 3];
    for (int i = blockIdx.x * kBlock + threadIdx.x; i < np; i += gridDim.x * kBlock)
      *hk_res(a, t, Lp[i]) = 0.0;
  }
  if (last_block(&c->done[DONE_DENSE], s_last, false) && threadIdx.x == 0) {
    if (MODE == kModeHK) {
      c->hk_tlc[0] = 0;
      c->hk_tlc[1] = 0;
      c->hk_tlc[2] = 0;
    } else if (dense_fuses<MODE>(c, t)) {
      c->cnt[(t + 1) & 1] = 0;  // what the self step listed is counted again by its row
    }
    c->cd_dirty |= 1 << (t & 1);
    if (c->dsteps == 0) c->pairs0 = c->steps;
    c->dense = DN_READY;
  }
}

__device__ __forceinline__ bool dense_wanted(const PlainArgs& a, const Ctl* c, int t,
                                             long long E) {
  return dense_pays(a, E) && !((c->cd_dirty >> (t & 1)) & 1);
}

// The self launch of PR-Nibble.  A frontier of at most one scan block goes
// to loop_rounds, run by workgroup 0; the others leave (counting them out would
// be 256 additions to one word at ~10 ns each).
__global__ __launch_bounds__(kSelfBlk) void k_self(PlainArgs a, int slot) {
  Ctl* c = a.ctl;
  const CtlHead h = ctl_head(c);
  if (h.dense != DN_LIST) return;  // k_dense's
  const int32_t nf = h.nf();
  if (h.status == ST_PUSH && nf > 0 && nf <= kScanBlock && h.round < h.max_rounds &&
      h.beta >= 1.0) {
    if (blockIdx.x == 0) loop_rounds(a, slot, h.round, nf);
    return;
  }
  self_body<kModePR, false, kSelfBlk>(a, slot, h);
}
__global__ __launch_bounds__(kBlock) void k_hk_self(PlainArgs a) {
  const CtlHead h = ctl_head(a.ctl);
  if (h.dense == DN_LIST) self_body<kModeHK, false, kBlock>(a, -1, h);
}
__global__ __launch_bounds__(kBlock) void k_nb_self(PlainArgs a) {
  self_body<kModeNB, false, kBlock>(a, -1, ctl_head(a.ctl));
}
// The entries of a round that the dense form has handed back.
__global__ __launch_bounds__(kBlock) void k_light_self(PlainArgs a, int slot) {
  const CtlHead h = ctl_head(a.ctl);
  if (h.dense == DN_LIGHT) self_body<kModePR, true, kBlock>(a, slot, h);
}
__global__ __launch_bounds__(kBlock) void k_hk_light_self(PlainArgs a) {
  const CtlHead h = ctl_head(a.ctl);
  if (h.dense == DN_LIGHT) self_body<kModeHK, true, kBlock>(a, -1, h);
}

// ------------------------------------------------- binned edge scatter
//
// For a large round, one FP64 atomic per edge is bound by contention on the
// lines of high-degree destinations.  The binned form of the same edgeMap
// (Figs. alg:pr-nibble / alg:pr-nibble2, UpdateNgh) groups the round's
// (neighbour, entry) pairs by destination bin, adds each bin's contributions
// in LDS and applies one update per distinct destination:
//   pass A (in k_scatter): every chunk of kBinChunk consecutive edges is
//     sorted by bin in place (a counting sort: LDS histogram with ranks, one
//     workgroup scan) into bin_pairs[chunk], and the start of every bin's run
//     in the chunk goes to bin_T (bin-major).  No global atomics.
//   pass B (k_bin_apply): one item per bin, or per slice of the chunks for a
//     bin whose expected share of the round's edges exceeds kBinQ.  The item
//     gathers its runs, adds every contribution into an LDS array over the
//     bin's vertex range (first touches listed), then updates each touched
//     destination once: a plain read-modify-write of r when the item owns the
//     whole bin (no other workgroup writes those records in this launch), a
//     device-scope atomic when the bin is split.  The filter is folded in as
//     in the atomic scatter: r only grows, so w joins the next frontier when
//     its single update (old, old + sum) straddles eps d(w).
// The sum of a destination's contributions is formed in another order than
// in a sequence of atomics; that is the only difference.

// LDS of the scatter launch: the atomic scatter's arrays or pass A's, which
// never run in the same launch.
struct ScatterLds {
  int32_t start[kEdgeTile + 1];
  int64_t row[kEdgeTile + 1];
  double coef[kEdgeTile + 1];
  __align__(8) unsigned short own[kEdgeTile];
  int32_t fn[kEdgeTile];
  int32_t tv[kEdgeTile];
  int nfn, ntv, base[2], last;
};
struct BinSortLds {
  int32_t start[kEdgeTile + 1];
  int64_t row[kEdgeTile + 1];
  int hist[kMaxBins + kBlock];
  int sh[kBlock / 64 + 1];
};
struct NbLds {
  int32_t fn[kBlock], tv[kBlock];
  int nfn, ntv, base[2];
};
union ScatterShared {
  ScatterLds at;
  BinSortLds bs;
  NbLds nb;
};

__device__ __forceinline__ bool bin_round(const PlainArgs& a, long long E) {
  return a.nbins > 0 && E >= a.bin_emin && E <= (long long)a.bin_cmax * kBinChunk;
}

// Exclusive scan over the workgroup of one int per thread; sh holds
// kBlock/64 + 1 slots.  Every thread must call it.
__device__ __forceinline__ int block_excl_scan_int(int x, int* total, int* sh) {
  int inc = x;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int y = __shfl_up(inc, o);
    if ((int)PLC_LANE >= o) inc += y;
  }
  if (PLC_LANE == 63) sh[PLC_WID] = inc;
  __syncthreads();
  if (threadIdx.x == 0) {
    int acc = 0;
    for (int w = 0; w < kBlock / 64; w++) {
      const int v = sh[w];
      sh[w] = acc;
      acc += v;
    }
    sh[kBlock / 64] = acc;
  }
  __syncthreads();
  const int ex = inc - x + sh[PLC_WID];
  *total = sh[kBlock / 64];
  __syncthreads();
  return ex;
}

// Pass A, run by the scatter launch in place of the atomic scatter.
// Workgroups take chunks in turn; a chunk's kBinChunkTiles tiles are staged
// one at a time (entries in LDS, a binary search per edge as in the atomic
// scatter).  The chunk's pairs stay in registers until the histogram scan.
__device__ void bin_sort_chunks(const PlainArgs& a, int nf, BinSortLds& L) {
  Ctl* c = a.ctl;
  int32_t* const s_start = L.start;
  int64_t* const s_row = L.row;
  int* const s_hist = L.hist;
  int* const sh = L.sh;
  constexpr int kPer = kBinChunk / kBlock;           // edges per thread per chunk
  constexpr int kBinsPT = kMaxBins / kBlock;         // bins per thread in the scan
  const int nb = a.nbins;
  const long long E = c->etotal;
  const int ntiles = (int64_t)c->ntiles > a.tile_cap ? (int)a.tile_cap : c->ntiles;
  const int C = (int)((E + kBinChunk - 1) / kBinChunk);
  for (int ch = blockIdx.x; ch < C; ch += gridDim.x) {
    for (int b = threadIdx.x; b < nb; b += kBlock) s_hist[b] = 0;
    __syncthreads();
    int32_t w[kPer], ie[kPer], bk[kPer];  // bk: bin << 16 | rank within the chunk's bin
#pragma unroll
    for (int tt = 0; tt < kBinChunkTiles; tt++) {
      const int tile = ch * kBinChunkTiles + tt;
      const long long e0 = (long long)tile * kEdgeTile;
      const long long e1 = e0 + kEdgeTile < E ? e0 + kEdgeTile : E;
      int cnt = 0, i0 = 0;
      if (tile < ntiles) {
        i0 = a.tile_start[tile];
        const int i1 = tile + 1 < ntiles ? a.tile_start[tile + 1] : nf - 1;
        cnt = i1 - i0 + 1;
        if (i0 < 0 || i1 < i0 || i1 >= nf || cnt > kEdgeTile + 1) {
          c->fault = 1;  // inconsistent tile map: the tile is skipped, the fault reported
          cnt = 0;
        }
        for (int j = threadIdx.x; j < cnt; j += kBlock) {
          s_start[j] = (int32_t)(a.estart[i0 + j] - e0);
          s_row[j] = a.rowp[i0 + j];
        }
      }
      __syncthreads();
#pragma unroll
      for (int k = 0; k < kEdgesPerThread; k++) {
        const int rel = k * kBlock + (int)threadIdx.x;
        const int x = tt * kEdgesPerThread + k;
        w[x] = -1;
        ie[x] = 0;
        if (cnt > 0 && e0 + rel < e1) {
          int lo = 0, hi = cnt - 1;
          while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (s_start[mid] <= rel) lo = mid; else hi = mid - 1;
          }
          w[x] = a.nbr[s_row[lo] + (rel - s_start[lo])];
          ie[x] = i0 + lo;
        }
      }
#pragma unroll
      for (int k = 0; k < kEdgesPerThread; k++) {
        const int x = tt * kEdgesPerThread + k;
        bk[x] = 0;
        if (w[x] >= 0) {
          const int b = a.bin_of_blk[w[x] / kBinGran];
          bk[x] = (b << 16) | atomicAdd(&s_hist[b], 1);
        }
      }
      __syncthreads();  // before the next tile's entries are staged
    }
    // run starts: exclusive prefix of the histogram (kBinsPT bins per thread)
    int loc[kBinsPT];
    int tsum = 0;
#pragma unroll
    for (int k = 0; k < kBinsPT; k++) {
      const int b = (int)threadIdx.x * kBinsPT + k;
      loc[k] = b < nb ? s_hist[b] : 0;
      tsum += loc[k];
    }
    int total;
    int ex = block_excl_scan_int(tsum, &total, sh);
#pragma unroll
    for (int k = 0; k < kBinsPT; k++) {
      const int b = (int)threadIdx.x * kBinsPT + k;
      if (b <= nb) {
        s_hist[b] = ex;
        a.bin_T[(size_t)b * a.bin_cmax + ch] = ex;
      }
      ex += loc[k];
    }
    __syncthreads();
    int2* out = a.bin_pairs + (size_t)ch * kBinChunk;
#pragma unroll
    for (int x = 0; x < kPer; x++) {
      if (w[x] >= 0) out[s_hist[bk[x] >> 16] + (bk[x] & 0xffff)] = make_int2(w[x], ie[x]);
    }
    __syncthreads();
  }
}

// Pass B of a binned round, then the round's close (exits at once when the
// round was not binned; k_scatter then closed it).  Each item gathers its
// bin's runs of (neighbour, entry) pairs from pass A and adds the entries'
// coefficients into an LDS array over the bin's vertices.  Then every touched
// destination gets one update (plain when the item owns the whole bin, atomic
// otherwise), on which its threshold crossing and first touch are decided.
template <int MODE>
__global__ __launch_bounds__(kBlock) void k_bin_apply(PlainArgs a, int slot) {
  Ctl* c = a.ctl;
  if (c->status != ST_PUSH) return;
  const int t = c->round;
  int nf = c->cnt[t & 1];
  if (nf <= 0) return;
  if ((int64_t)nf > a.n) nf = (int)a.n;
  if (t >= c->max_rounds || c->selfed != t || c->dense != DN_LIST) return;
  const long long E = c->etotal;
  if (!bin_round(a, E)) return;
  __shared__ double acc[kBinWidth];          // the item's sums, zero between items
  __shared__ int32_t s_list[kBinWidth];      // first touches of the item (offsets in the bin)
  __shared__ int s_items[kMaxBins + 1];      // first item of each bin
  // start of the item's run in each chunk, and the exclusive prefix of the
  // run lengths
  __shared__ int s_rs[kBinItemChunks], s_rp[kBinItemChunks];
  __shared__ int sh[kBlock / 64 + 1];
  __shared__ int s_nl, s_fb, s_tb, s_last;
  constexpr int kBinsPT = kMaxBins / kBlock;
  constexpr int kRunsPT = kBinItemChunks / kBlock;
  constexpr int kListPT = kBinWidth / kBlock;
  static_assert(kListPT <= 32, "flush masks are 32 bits");
  static_assert(kBinWidth < 65536, "the flush packs two counts in one int");
  const int nb = a.nbins;
  const int C = (int)((E + kBinChunk - 1) / kBinChunk);
  const double eps = c->eps;
  int32_t* Fn = (t & 1) ? a.fbuf0 : a.fbuf1;
  int32_t* cntn = &c->cnt[(t + 1) & 1];
  // where first touches go
  constexpr bool NB = MODE == kModeNB;
  const int list = (t + 1) % 3;
  int32_t* const tv_list = NB ? a.hk_tl[list] : a.touched;
  int32_t* const tv_cnt = NB ? &c->hk_tlc[list] : &c->touched_cnt;
  for (int j = threadIdx.x; j < kBinWidth; j += kBlock) acc[j] = 0.0;
  // items per bin: the bin's expected share of the round's edges (E vol_b /
  // 2m) over kBinQ, at least enough that an item spans <= kBinItemChunks
  // chunks, at most one per chunk; every workgroup computes the same table
  {
    const int smin = (C + kBinItemChunks - 1) / kBinItemChunks;
    int loc[kBinsPT];
    int tsum = 0;
#pragma unroll
    for (int k = 0; k < kBinsPT; k++) {
      const int b = (int)threadIdx.x * kBinsPT + k;
      int it = 0;
      if (b < nb) {
        const double expect = (double)E * (double)a.bin_vol[b] / (double)a.vol_total;
        it = (int)ceil(expect / (double)kBinQ);
        it = it > smin ? it : smin;
        it = it < C ? it : C;
        it = it > 1 ? it : 1;
      }
      loc[k] = it;
      tsum += it;
    }
    int total;
    int ex = block_excl_scan_int(tsum, &total, sh);
#pragma unroll
    for (int k = 0; k < kBinsPT; k++) {
      const int b = (int)threadIdx.x * kBinsPT + k;
      if (b < nb) s_items[b] = ex;
      ex += loc[k];
    }
    if (threadIdx.x == 0) {
      s_items[nb] = total;
      s_nl = 0;
    }
    __syncthreads();
  }
  const int items = s_items[nb];
  for (int it = blockIdx.x; it < items; it += gridDim.x) {
    int lo = 0, hi = nb - 1;  // the bin: last b with s_items[b] <= it
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (s_items[mid] <= it) lo = mid; else hi = mid - 1;
    }
    const int b = lo;
    const int S = s_items[b + 1] - s_items[b];
    const int sl = it - s_items[b];
    const int vlo = a.bin_lo[b];
    const int W = a.bin_lo[b + 1] - vlo;
    const bool own = S == 1;
    const int c0 = (int)((long long)sl * C / S), c1 = (int)((long long)(sl + 1) * C / S);
    const int nc = c1 - c0;
    // the item's runs
    int rl[kRunsPT];
    int lsum = 0;
#pragma unroll
    for (int k = 0; k < kRunsPT; k++) {
      const int q = (int)threadIdx.x * kRunsPT + k;
      rl[k] = 0;
      if (q < nc) {
        const int st = a.bin_T[(size_t)b * a.bin_cmax + c0 + q];
        const int en = a.bin_T[(size_t)(b + 1) * a.bin_cmax + c0 + q];
        s_rs[q] = (c0 + q) * kBinChunk + st;
        rl[k] = en - st;
        if (rl[k] < 0 || en > kBinChunk) { c->fault = 1; rl[k] = 0; }
      }
      lsum += rl[k];
    }
    int L;
    int ex = block_excl_scan_int(lsum, &L, sh);
#pragma unroll
    for (int k = 0; k < kRunsPT; k++) {
      const int q = (int)threadIdx.x * kRunsPT + k;
      if (q < nc) s_rp[q] = ex;
      ex += rl[k];
    }
    __syncthreads();
    // add every contribution into the LDS array; the first toucher of an
    // offset lists it
    constexpr int kU = 4;
    for (int j0 = 0; j0 < L; j0 += kBlock * kU) {
      int2 pr[kU];
#pragma unroll
      for (int u = 0; u < kU; u++) {
        const int j = j0 + u * kBlock + (int)threadIdx.x;
        pr[u] = make_int2(-1, 0);
        if (j < L) {
          int l2 = 0, h2 = nc - 1;
          while (l2 < h2) {
            const int mid = (l2 + h2 + 1) >> 1;
            if (s_rp[mid] <= j) l2 = mid; else h2 = mid - 1;
          }
          pr[u] = a.bin_pairs[s_rs[l2] + (j - s_rp[l2])];
        }
      }
      double cf[kU];
#pragma unroll
      for (int u = 0; u < kU; u++) cf[u] = pr[u].x >= 0 && pr[u].y < nf ? a.coef[pr[u].y] : 0.0;
#pragma unroll
      for (int u = 0; u < kU; u++) {
        const int jl = pr[u].x - vlo;
        bool first = false;
        if (pr[u].x >= 0) {
          // (contributions are positive, so exactly one addition per touched
          // offset returns 0; an impossible zero one is not listed)
          if (jl >= 0 && jl < W) first = atomicAdd(&acc[jl], cf[u]) == 0.0 && cf[u] != 0.0;
          else c->fault = 1;
        }
        wave_append(first, jl, s_list, &s_nl);
      }
    }
    __syncthreads();
    // one update per touched destination
    const int nl = s_nl;
    unsigned fm = 0, tm = 0;
    int nfl = 0, ntl = 0;
    int32_t jv[kListPT];
    double xv[kListPT];
#pragma unroll
    for (int m = 0; m < kListPT; m++) {
      const int k = m * kBlock + (int)threadIdx.x;
      jv[m] = -1;
      xv[m] = 0.0;
      if (k < nl) {
        jv[m] = s_list[k];
        xv[m] = acc[jv[m]];
        acc[jv[m]] = 0.0;
      }
    }
#pragma unroll
    for (int m = 0; m < kListPT; m++) {
      if (jv[m] < 0) continue;
      const int32_t w = vlo + jv[m];
      double old, thr;
      if (own && !NB) {
        const VRec rec = a.vr[w];
        old = rec.r;
        a.vr[w].r = old + xv[m];
        thr = eps * (double)rec.deg;
      } else {
        double* const dst = NB ? hk_res(a, t + 1, w) : &a.vr[w].r;
        thr = eps * (double)a.vr[w].deg;
        if (own) {
          old = *dst;
          *dst = old + xv[m];
        } else {
          old = unsafeAtomicAdd(dst, xv[m]);
        }
      }
      if (old < thr && old + xv[m] >= thr) { fm |= 1u << m; nfl++; }
      if (__double_as_longlong(old) == 0) { tm |= 1u << m; ntl++; }
    }
    // both counts in one scan (each total is at most kBinWidth < 2^16)
    int both;
    const int bex = block_excl_scan_int(nfl | (ntl << 16), &both, sh);
    const int fex = bex & 0xffff, tex = bex >> 16;
    const int NF = both & 0xffff, NT = both >> 16;
    if (threadIdx.x == 0) {
      s_fb = NF > 0 ? atomicAdd(cntn, NF) : 0;
      s_tb = NT > 0 ? atomicAdd(tv_cnt, NT) : 0;
      s_nl = 0;
    }
    __syncthreads();
    long long pf = (long long)s_fb + fex, pt = (long long)s_tb + tex;
#pragma unroll
    for (int m = 0; m < kListPT; m++) {
      if (jv[m] < 0) continue;
      const int32_t w = vlo + jv[m];
      if (fm >> m & 1u) {
        if (pf < a.n) Fn[pf] = w; else c->fault = 1;
        pf++;
      }
      if (tm >> m & 1u) {
        if (pt < a.n) tv_list[pt] = w; else c->fault = 1;
        pt++;
      }
    }
    __syncthreads();
  }
  if (last_block(&c->done[DONE_BIN], &s_last, false)) {
    if (threadIdx.x == 0) {
      c->pushes += nf;
      c->edges += E;
      c->bin_rounds += 1;
      c->bin_edges += E;
      c->cnt[t & 1] = 0;
      c->round = t + 1;
      if (slot >= 0) a.work_log[2 * slot + 1] = 1;
    }
  }
}

// The kept halves of a binned Nibble step, added before pass B (a launch of
// its own) adds the contributions: an entry's vertex gets h = rho / 2.  20 steps
// of up to 6 M edges (R-MAT 2^22, eps 1e-8) take 37 us each in pass A, the
// halves included, and 70 in pass B; with one atomic per edge 189.
__device__ void nb_halves(const PlainArgs& a, int t, int nf, double eps, NbLds& L) {
  Ctl* c = a.ctl;
  const int32_t* Fc = (t & 1) ? a.fbuf1 : a.fbuf0;
  int32_t* Fn = (t & 1) ? a.fbuf0 : a.fbuf1;
  const int list = (t + 1) % 3;
  if (threadIdx.x == 0) {
    L.nfn = 0;
    L.ntv = 0;
  }
  __syncthreads();
  for (int b0 = blockIdx.x * kBlock; b0 < nf; b0 += gridDim.x * kBlock) {
    const int i = b0 + (int)threadIdx.x;
    if (i < nf) {
      const int32_t v = Fc[i];
      const double h = a.sp[i];
      const double thr = eps * (double)a.vr[v].deg;
      const double o = unsafeAtomicAdd(hk_res(a, t + 1, v), h);
      decide(true, o, h, thr, v, L.fn, &L.nfn, L.tv, &L.ntv);
    }
    block_flush2(&c->cnt[(t + 1) & 1], Fn, L.fn, &L.nfn, &c->hk_tlc[list], a.hk_tl[list], L.tv,
                 &L.ntv, a.n, L.base, &c->fault);
  }
}

// edgeMap(G, Frontier, UpdateNgh) with the filter folded in.  Each
// workgroup takes a contiguous range of edge tiles; every edge is one
// device-scope FP64 atomic.  (Combining the contributions to the
// highest-degree destinations in LDS, as the batched scatter does, measured
// slower here: one query's round spreads over few workgroups, and the
// per-workgroup clear and flush cost more than the contention they save.)
//   PR-Nibble: into r, threshold eps d(w), first touches to the touched list.
//   HK-PR level j: into the level-(j+1) residuals, threshold
//     ((e^-t eps) d(w)) / (2 N psi_{j+1}), first touches to level j+1's list;
//     on the last level into p (UpdateNghLast), first touches of p to the
//     support list, no frontier.
//   Nibble step j -> j+1: into vector j+1, threshold eps d(w), first touches
//     to list j+1; each entry's own rho / 2 is added by the workgroup whose
//     tile holds the entry's first edge.
template <int MODE>
__device__ __forceinline__ void scatter_body(const PlainArgs& a, int slot, ScatterShared& sm,
                                             int pair = -1, bool apply = true) {
  constexpr bool HK = MODE == kModeHK;
  constexpr bool LEVELS = MODE != kModePR;
  Ctl* c = a.ctl;
  CtlEdges q;
  const CtlHead h = ctl_head(c, &q);
  int t, nf;
  if (MODE == kModePR && blockIdx.x == 0 && threadIdx.x == 0 && h.nf() == 0 && c->pend > 0) {
    c->cnt[h.round & 1] = c->pend;  // (no entries yet: every workgroup leaves below)
    c->pend = 0;
  }
  if (!push_active(h, a.n, &t, &nf)) return;
  if (h.selfed != t) return;  // no entries built for this round (a self loop stopped before it)
  if (MODE != kModeNB && h.dense != DN_LIST) return;  // k_dense's
  if (t >= (HK ? c->hk_N : h.max_rounds)) return;
  if (MODE != kModeNB && dense_wanted(a, c, t, q.etotal)) {
    dense_enter<MODE>(a, t, nf, &sm.at.last);
    return;
  }
  // which launch pairs of a first chunk carry rounds that could bin (the
  // host queues k_bin_apply behind those pairs only); without k_bin_apply
  // behind it such a round takes the atomic form
  // (Nibble: which steps could bin)
  if (!HK && bin_round(a, q.etotal)) {
    if (MODE == kModeNB) pair = t < 31 ? t : 31;
    if (pair >= 0 && blockIdx.x == 0 && threadIdx.x == 0) c->bin_pairs |= 1u << pair;
    if (apply) {
      bin_sort_chunks(a, nf, sm.bs);  // pass A; k_bin_apply adds and closes the round
      if (MODE == kModeNB) nb_halves(a, t, nf, q.eps, sm.nb);
      return;
    }
  }
  int32_t* const s_start = sm.at.start;
  int64_t* const s_row = sm.at.row;
  double* const s_coef = sm.at.coef;
  int32_t* const s_fn = sm.at.fn;
  int32_t* const s_tv = sm.at.tv;
  int& s_nfn = sm.at.nfn;
  int& s_ntv = sm.at.ntv;
  int* const s_base = sm.at.base;
  int& s_last = sm.at.last;
  const int ntiles = (int64_t)q.ntiles > a.tile_cap ? (int)a.tile_cap : q.ntiles;
  const long long E = q.etotal;
  const bool hk_last = HK && t + 1 == c->hk_N;
  const double eps = HK ? c->hk_A : q.eps;                    // threshold numerator factor
  const int32_t* Fc = (t & 1) ? a.fbuf1 : a.fbuf0;            // this round's frontier
  const double den = HK && !hk_last ? a.hk_B[t + 1] : 1.0;    // threshold denominator
  int32_t* Fn = (t & 1) ? a.fbuf0 : a.fbuf1;
  int32_t* cntn = &c->cnt[(t + 1) & 1];
  // where first touches go
  int32_t* tv_list = LEVELS ? (hk_last ? a.support : a.hk_tl[(t + 1) % 3]) : a.touched;
  int32_t* tv_cnt =
      LEVELS ? (hk_last ? &c->support_cnt : &c->hk_tlc[(t + 1) % 3]) : &c->touched_cnt;
  const int per = (ntiles + gridDim.x - 1) / gridDim.x;
  const int tb = blockIdx.x * per;
  const int te = tb + per < ntiles ? tb + per : ntiles;
  // workgroups without tiles (large grids, small rounds) leave at once; the
  // round is closed by the last of the `busy` ones (at least workgroup 0)
  const int busy = per > 0 ? (ntiles + per - 1) / per : 1;
  if ((int)blockIdx.x >= busy) return;
  if (threadIdx.x == 0) { s_nfn = 0; s_ntv = 0; }
  __syncthreads();

  for (int tile = tb; tile < te; tile++) {
    const long long e0 = (long long)tile * kEdgeTile;
    const long long e1 = e0 + kEdgeTile < E ? e0 + kEdgeTile : E;
    const int i0 = a.tile_start[tile];
    const int i1 = tile + 1 < ntiles ? a.tile_start[tile + 1] : nf - 1;
    if (i0 < 0 || i1 < i0 || i1 >= nf || i1 - i0 + 1 > kEdgeTile + 1) {
      c->fault = 1;  // inconsistent tile map: skip the tile, report a fault
      continue;
    }
    const int cnt = i1 - i0 + 1;
    for (int j = threadIdx.x; j < cnt; j += kBlock) {
      s_start[j] = (int32_t)(a.estart[i0 + j] - e0);
      s_row[j] = a.rowp[i0 + j];
      s_coef[j] = a.coef[i0 + j];
    }
    __syncthreads();
    // The entry of every edge: each thread searches for the first of four
    // consecutive edges and walks on from it.  The edges are then taken
    // kBlock apart, so that a wave's 64 neighbours are consecutive (their
    // loads, and the atomics on records of one line, go out together).
    const int len = (int)(e1 - e0);
    {
      const int r0 = (int)threadIdx.x * kEdgesPerThread;
      int lo = 0, hi = cnt - 1;
      while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (s_start[mid] <= r0) lo = mid; else hi = mid - 1;
      }
      ushort4 at;
      at.x = lo;
      // (every entry has an edge, so the next edge is at most one entry on)
      if (lo + 1 < cnt && s_start[lo + 1] <= r0 + 1) lo++;
      at.y = lo;
      if (lo + 1 < cnt && s_start[lo + 1] <= r0 + 2) lo++;
      at.z = lo;
      if (lo + 1 < cnt && s_start[lo + 1] <= r0 + 3) lo++;
      at.w = lo;
      static_assert(kEdgesPerThread == 4 && kEdgeTile < 65536, "four 16-bit entries");
      reinterpret_cast<ushort4*>(sm.at.own)[threadIdx.x] = at;
    }
    __syncthreads();
    // Four independent edges per thread: all neighbour loads, then all
    // degree loads and atomics, then the decisions, so latencies overlap.
    int32_t w[kEdgesPerThread];
    double cf[kEdgesPerThread];
#pragma unroll
    for (int k = 0; k < kEdgesPerThread; k++) {
      const int rel = k * kBlock + (int)threadIdx.x;
      const int at = sm.at.own[rel];
      w[k] = rel < len ? a.nbr[s_row[at] + (rel - s_start[at])] : -1;
      cf[k] = s_coef[at];
    }
    int32_t dw[kEdgesPerThread];
#pragma unroll
    for (int k = 0; k < kEdgesPerThread; k++) dw[k] = w[k] >= 0 && !hk_last ? a.vr[w[k]].deg : 0;
    double old[kEdgesPerThread];
#pragma unroll
    for (int k = 0; k < kEdgesPerThread; k++) {
      double* dst = nullptr;
      if (w[k] >= 0) dst = !LEVELS ? &a.vr[w[k]].r : hk_last ? &a.p[w[k]] : hk_res(a, t + 1, w[k]);
      old[k] = dst ? unsafeAtomicAdd(dst, cf[k]) : 0.0;
    }
    unsigned cross = 0, touch = 0;  // bit k: edge k
#pragma unroll
    for (int k = 0; k < kEdgesPerThread; k++) {
      const double thr = (eps * (double)dw[k]) / den;
      if (w[k] < 0) continue;
      if (!hk_last && old[k] < thr && old[k] + cf[k] >= thr) cross |= 1u << k;
      if (first_touch(old[k], cf[k])) touch |= 1u << k;
    }
    if (!hk_last) wave_append_all<kEdgesPerThread>(cross, w, s_fn, &s_nfn);
    wave_append_all<kEdgesPerThread>(touch, w, s_tv, &s_ntv);
    block_flush2(cntn, Fn, s_fn, &s_nfn, tv_cnt, tv_list, s_tv, &s_ntv, a.n, s_base, &c->fault);
    if (MODE == kModeNB) {
      // the kept halves of the entries whose first edge is in this tile
      for (int jj = threadIdx.x; jj < cnt; jj += kBlock) {
        const int st = s_start[jj];
        if (st < 0 || e0 + st >= e1) continue;
        const int i = i0 + jj;
        const int32_t v = Fc[i];
        const double h = a.sp[i];
        const double o = unsafeAtomicAdd(hk_res(a, t + 1, v), h);
        decide(true, o, h, eps * (double)a.vr[v].deg, v, s_fn, &s_nfn, s_tv, &s_ntv);
      }
      block_flush2(cntn, Fn, s_fn, &s_nfn, tv_cnt, tv_list, s_tv, &s_ntv, a.n, s_base, &c->fault);
    }
  }
  if (last_block_of(&c->done[DONE_SCATTER], &s_last, false, (unsigned)busy)) {
    if (threadIdx.x == 0) {
      c->pushes += nf;
      c->edges += E;
      c->cnt[t & 1] = 0;
      c->round = t + 1;
      if (slot >= 0) a.work_log[2 * slot + 1] = 1;
    }
  }
}

__global__ __launch_bounds__(kBlock) void k_scatter(PlainArgs a, int slot, int pair, int apply) {
  __shared__ ScatterShared sm;
  scatter_body<kModePR>(a, slot, sm, pair, apply != 0);
}
__global__ __launch_bounds__(kBlock) void k_hk_scatter(PlainArgs a) {
  __shared__ ScatterShared sm;
  scatter_body<kModeHK>(a, -1, sm);
}
__global__ __launch_bounds__(kBlock) void k_nb_scatter(PlainArgs a, int apply) {
  __shared__ ScatterShared sm;
  scatter_body<kModeNB>(a, -1, sm, -1, apply != 0);
}

// HK-PR initialisation (Fig. alg:hkpr: r = {(x, 1)}, Frontier = {x},
// j = 0); level 0 touched only x.
__global__ void k_hk_init(PlainArgs a, int32_t x, int32_t N, double t, double A) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  Ctl* c = a.ctl;
  c->cs = 0.0;
  c->cn = 0.0;
  c->keep = 0.0;
  c->eps = 0.0;
  c->seed = x;
  c->rule = -1;
  c->max_rounds = N;
  c->opt_rule = 1;
  c->round = 0;
  c->cnt[0] = 1;
  c->cnt[1] = 0;
  c->ntiles = 0;
  c->etotal = 0;
  c->pushes = 0;
  c->edges = 0;
  c->support_cnt = 0;
  c->touched_cnt = 0;  // no residual is reported: the sweep gathers none
  c->fault = 0;
  c->limited = 0;
  c->N = 0;
  c->sort_flip = 0;
  c->rnnz = 0;
  c->vol_total = a.vol_total;
  c->best_cut = 0;
  c->best_vol = 0;
  c->best_den = 0;
  c->kstar = 0;
  c->phi = 0.0;
  reset_round_book(c);
  c->hk_N = N;
  c->hk_t = t;
  c->hk_A = A;
  c->hk_tlc[0] = 1;
  c->hk_tlc[1] = 0;
  c->hk_tlc[2] = 0;
  a.hk_tl[0][0] = x;
  a.fbuf0[0] = x;
  a.vr[x].r = 1.0;
  c->status = ST_PUSH;
}

// Nibble initialisation (Fig. alg:nibble: p = {(x, 1)}, Frontier = {x});
// vector 0 is the seed's indicator, its support list holds x.
__global__ void k_nb_init(PlainArgs a, int32_t x, double eps, int32_t T) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  Ctl* c = a.ctl;
  c->cs = 0.0;
  c->cn = 0.0;
  c->keep = 0.0;
  c->eps = eps;
  c->seed = x;
  c->rule = -2;
  c->max_rounds = T;
  c->opt_rule = 1;
  c->round = 0;
  c->cnt[0] = 1;
  c->cnt[1] = 0;
  c->ntiles = 0;
  c->etotal = 0;
  c->pushes = 0;
  c->edges = 0;
  c->support_cnt = 0;
  c->touched_cnt = 0;
  c->fault = 0;
  c->limited = 0;
  c->N = 0;
  c->sort_flip = 0;
  c->rnnz = 0;
  c->vol_total = a.vol_total;
  c->best_cut = 0;
  c->best_vol = 0;
  c->best_den = 0;
  c->kstar = 0;
  c->phi = 0.0;
  reset_round_book(c);
  c->hk_N = 0;
  c->hk_tlc[0] = 1;
  c->hk_tlc[1] = 0;
  c->hk_tlc[2] = 0;
  a.hk_tl[0][0] = x;
  a.fbuf0[0] = x;
  a.vr[x].r = 1.0;
  c->status = ST_PUSH;
}

// End of Nibble after J steps, returning vector R (J, or J - 1 when step J
// left an empty frontier): p and the support list take vector R over the
// vertices it touched, and both vector arrays are cleared (vector J over
// list J, vector J - 1 over list J - 1: every earlier one was cleared by
// the self kernel two steps later; each entry of vector R is read and
// cleared by the same thread).  The frontier count is zeroed so that the
// sweep may start.
__global__ __launch_bounds__(kBlock) void k_nb_finish(PlainArgs a, int32_t R, int32_t J) {
  Ctl* c = a.ctl;
  for (int q = 0; q < 2; q++) {
    const int lv = J - q;
    if (lv < 0) continue;
    const int li = lv % 3;
    const int cnt = c->hk_tlc[li];
    const int32_t* L = a.hk_tl[li];
    for (int i = blockIdx.x * kBlock + threadIdx.x; i < cnt; i += gridDim.x * kBlock) {
      const int32_t v = L[i];
      double* x = hk_res(a, lv, v);
      if (lv == R) {
        a.p[v] = *x;
        a.support[i] = v;
      }
      *x = 0.0;
    }
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    c->support_cnt = c->hk_tlc[R % 3];
    c->cnt[J & 1] = 0;
  }
}

// After the last HK-PR level (nothing before it): residuals can remain only
// on the vertices the last two levels touched (every earlier level was
// cleared by the self kernel two levels later, and the dense form keeps
// none); clear both arrays there.
__global__ __launch_bounds__(kBlock) void k_hk_clear(PlainArgs a) {
  Ctl* c = a.ctl;
  const int J = c->round;
  if (c->cnt[J & 1] > 0 && J < c->hk_N) return;
  for (int q = 0; q < 2; q++) {
    const int lv = J - q;
    if (lv < 0) continue;
    const int li = lv % 3;
    const int cnt = c->hk_tlc[li];
    const int32_t* L = a.hk_tl[li];
    for (int i = blockIdx.x * kBlock + threadIdx.x; i < cnt; i += gridDim.x * kBlock) {
      const int32_t v = L[i];
      a.vr[v].r = 0.0;
      a.hk_r1[v] = 0.0;
    }
  }
}

// ---------------------------------------------------------------- beta variant
// PR-Nibble pushing the top beta fraction of the active set by r/d per round
// (end of Sec. 3.3).  The frontier holds the whole active set; before the
// round it is ranked with the sweep's sort (keys: bit-inverted r/d, ties by
// ascending id) and the top k = ceil(beta |F|) move to its front as the
// round's frontier; after the round the other |F| - k, still at or above
// their thresholds (their r only grew), join the next frontier.

// Sort keys of the active set (count in N; 0 when the push has ended).
__global__ __launch_bounds__(kBlock) void k_beta_keys(PlainArgs a) {
  Ctl* c = a.ctl;
  int t, nf;
  if (!push_active(ctl_head(c), a.n, &t, &nf) || t >= c->max_rounds) {
    if (blockIdx.x == 0 && threadIdx.x == 0) { c->N = 0; c->beta_nf = 0; }
    return;
  }
  const int32_t* F = (t & 1) ? a.fbuf1 : a.fbuf0;
  for (int i = blockIdx.x * kBlock + threadIdx.x; i < nf; i += gridDim.x * kBlock) {
    const int32_t v = F[i];
    const VRec rec = a.vr[v];
    SortElem e;
    e.key = ~(unsigned long long)__double_as_longlong(rec.r / (double)rec.deg);
    e.id = v;
    e.seg = 0;
    a.sbuf[0][i] = e;
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    c->N = nf;
    c->sort_flip = 0;
    c->beta_nf = nf;
  }
}

// Ranked active set back into the frontier buffer; the round's frontier is
// its first k entries.
__global__ __launch_bounds__(kBlock) void k_beta_select(PlainArgs a) {
  Ctl* c = a.ctl;
  const int nf = c->beta_nf;
  if (nf <= 0) return;
  const int t = c->round;
  int32_t* F = (t & 1) ? a.fbuf1 : a.fbuf0;
  const SortElem* el = a.sbuf[c->sort_flip & 1];
  for (int i = blockIdx.x * kBlock + threadIdx.x; i < nf; i += gridDim.x * kBlock) F[i] = el[i].id;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    long long k = (long long)ceil(c->beta * (double)nf);
    if (k < 1) k = 1;
    if (k > nf) k = nf;
    c->beta_k = (int32_t)k;
    c->cnt[t & 1] = (int32_t)k;
  }
}

// After the round: the unpushed part of the ranked set joins the next
// frontier (one counter atomic per workgroup step).
__global__ __launch_bounds__(kBlock) void k_beta_carry(PlainArgs a) {
  Ctl* c = a.ctl;
  const int nf = c->beta_nf, k = c->beta_k;
  if (nf <= k) return;
  const int t = c->round;              // the round just closed was t - 1
  const int32_t* F = ((t - 1) & 1) ? a.fbuf1 : a.fbuf0;
  int32_t* Fn = (t & 1) ? a.fbuf1 : a.fbuf0;
  __shared__ int s_base;
  for (int i0 = k + blockIdx.x * kBlock; i0 < nf; i0 += gridDim.x * kBlock) {
    const int m = nf - i0 < kBlock ? nf - i0 : kBlock;
    if (threadIdx.x == 0) s_base = atomicAdd(&c->cnt[t & 1], m);
    __syncthreads();
    if ((int)threadIdx.x < m) {
      const long long slot = (long long)s_base + threadIdx.x;
      if (slot < a.n) Fn[slot] = F[i0 + threadIdx.x]; else c->fault = 1;
    }
    __syncthreads();
  }
}

// ---------------------------------------------------------------- sweep

// The sweep may start once the frontier is empty (or the watchdog fired).
__device__ __forceinline__ bool sweep_ready(const Ctl* c) {
  const CtlHead h = ctl_head(c);
  return h.status == ST_LIMIT || (h.status == ST_PUSH && h.nf() == 0);
}

// Sort keys: non-increasing p/d is ascending order of the bit-inverted IEEE
// pattern of the positive ratio; equal ratios order by ascending id.
// The sweep sequence is queued for supports of at most `bound` vertices (it
// sets the sort's launches); a larger support leaves the query unswept, for
// a sweep queued with a larger bound.
__global__ __launch_bounds__(kBlock) void k_sweep_keys(PlainArgs a, long long bound) {
  Ctl* c = a.ctl;
  const int scnt = c->support_cnt;
  if (!sweep_ready(c) || (long long)scnt > bound) return;
  __shared__ int s_last;
  const int N = (int64_t)scnt > a.n ? (int)a.n : scnt;
  const int dirty = c->cd_dirty;
  // the workgroups that have keys to form (all, to clear the coefficients)
  const int want = (N + kBlock - 1) / kBlock;
  const int busy = dirty || want > (int)gridDim.x ? (int)gridDim.x : want > 1 ? want : 1;
  if ((int)blockIdx.x >= busy) return;
  for (int i = blockIdx.x * kBlock + threadIdx.x; i < N; i += busy * kBlock) {
    int32_t v = a.support[i];
    double ratio = a.p[v] / (double)a.vr[v].deg;
    SortElem e;
    e.key = ~(unsigned long long)__double_as_longlong(ratio);
    e.id = v;
    e.seg = 0;
    a.sbuf[0][i] = e;
  }
  // a push that ended in the dense form leaves its last coefficients
  for (int k = 0; k < 2; k++)
    if ((dirty >> k) & 1)
      for (int64_t i = blockIdx.x * kBlock + threadIdx.x; i < a.n; i += gridDim.x * kBlock)
        a.cd[k][i] = 0.0;
  if (last_block_of(&c->done[DONE_KEYS], &s_last, false, (unsigned)busy)) {
    if (threadIdx.x == 0) {
      c->N = N;
      c->sort_flip = 0;
      c->cd_dirty = 0;
      c->status = ST_SWEEPING;
    }
  }
}

// Rank map (rank[v_k] = k, outside = 0) with per-position degree, p and id,
// and the inclusive volume prefix vol(S_k) with the edge-tile map over the
// support's edges in sweep order (the offsets of the Z array in Theorem 1's
// proof).
__global__ __launch_bounds__(kBlock) void k_vol_scan(PlainArgs a) {
  Ctl* c = a.ctl;
  if (c->status != ST_SWEEPING) return;
  const int N = c->N;
  if (N <= 0) return;
  const SortElem* el = a.sbuf[c->sort_flip & 1];
  int32_t* const out_ids = a.sid;
  double* const out_p = a.sp;
  __shared__ long long sh[kBlock / 64 + 1];
  __shared__ long long s_excl;
  __shared__ unsigned long long s_tk;
  const int nblk = (N + kScanBlock - 1) / kScanBlock;
  const bool fixed = scan_fixed(nblk);
  if (fixed && (int)blockIdx.x >= nblk) return;
  ScanSite* site = &c->scan[SCAN_VOL];
  unsigned long long* desc;
  for (int b = scan_begin(site, a.desc[SCAN_VOL], a.desc_cap, nblk, fixed, &s_tk, &desc); b < nblk;
       b = scan_next(site, nblk, fixed, &s_tk)) {
    // kScanItems consecutive positions per thread (see k_self)
    const int i0 = b * kScanBlock + (int)threadIdx.x * kScanItems;
    int32_t dk[kScanItems];
    long long dsum = 0;
#pragma unroll
    for (int k = 0; k < kScanItems; k++) {
      const int i = i0 + k;
      dk[k] = 0;
      if (i < N) {
        const int32_t v = el[i].id;
        a.vr[v].rank = i + 1;
        dk[k] = a.vr[v].deg;
        a.sdeg[i] = dk[k];
        out_p[i] = a.p[v];
        out_ids[i] = v;
        a.scnt[i] = 0;
      }
      dsum += dk[k];
    }
    long long agg;
    const long long ex = block_excl_scan<kBlock>(dsum, &agg, sh);
    if (threadIdx.x < 64) {
      const long long ex0 = scan_lookback(desc, b, agg, &c->fault);
      if (threadIdx.x == 0) s_excl = ex0;
    }
    __syncthreads();
    long long s = s_excl + ex;
#pragma unroll
    for (int k = 0; k < kScanItems; k++) {
      const int i = i0 + k;
      if (i < N) {
        a.svol[i] = s + dk[k];
        mark_tiles(a.tile_start, a.tile_cap, s, dk[k], i, &c->fault);
      }
      s += dk[k];
    }
    if (b == nblk - 1 && threadIdx.x == 0) {
      const long long base = s_excl + agg;
      c->etotal = base;
      c->ntiles = (int)((base + kEdgeTile - 1) / kEdgeTile);
    }
    __syncthreads();
  }
}

// For every support edge (v_k, w): count w with 1 <= rank[w] < k.  Then
// delta_k = d(v_k) - 2 * count_k is the change of the boundary when v_k joins
// S_{k-1}; it equals the sum of Z's first values at rank k (Theorem 1).
__global__ __launch_bounds__(kBlock) void k_cut_count(PlainArgs a) {
  Ctl* c = a.ctl;
  if (c->status != ST_SWEEPING) return;
  const int N = c->N;
  if (N <= 0) return;
  __shared__ int32_t s_start[kEdgeTile + 1];
  __shared__ int64_t s_row[kEdgeTile + 1];
  __shared__ int32_t s_cnt[kEdgeTile + 1];
  const int32_t* const sid = a.sid;
  const int ntiles = (int64_t)c->ntiles > a.tile_cap ? (int)a.tile_cap : c->ntiles;
  const long long E = c->etotal;
  for (int tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
    const long long e0 = (long long)tile * kEdgeTile;
    const long long e1 = e0 + kEdgeTile < E ? e0 + kEdgeTile : E;
    const int i0 = a.tile_start[tile];
    const int i1 = tile + 1 < ntiles ? a.tile_start[tile + 1] : N - 1;
    if (i0 < 0 || i1 < i0 || i1 >= N || i1 - i0 + 1 > kEdgeTile + 1) {
      c->fault = 1;
      continue;
    }
    const int cnt = i1 - i0 + 1;
    for (int j = threadIdx.x; j < cnt; j += kBlock) {
      int k = i0 + j;
      s_start[j] = (int32_t)(a.svol[k] - a.sdeg[k] - e0);
      s_row[j] = a.off[sid[k]];
      s_cnt[j] = 0;
    }
    __syncthreads();
    int32_t rw[kEdgesPerThread];
    int own[kEdgesPerThread];
#pragma unroll
    for (int kk = 0; kk < kEdgesPerThread; kk++) {
      const int rel = kk * kBlock + (int)threadIdx.x;
      own[kk] = -1;
      rw[kk] = 0;
      if (e0 + rel < e1) {
        int lo = 0, hi = cnt - 1;
        while (lo < hi) {
          int mid = (lo + hi + 1) >> 1;
          if (s_start[mid] <= rel) lo = mid; else hi = mid - 1;
        }
        int32_t w = a.nbr[s_row[lo] + (rel - s_start[lo])];
        rw[kk] = a.vr[w].rank;
        own[kk] = lo;
      }
    }
#pragma unroll
    for (int kk = 0; kk < kEdgesPerThread; kk++) {
      if (own[kk] >= 0 && rw[kk] > 0 && rw[kk] < i0 + own[kk] + 1) atomicAdd(&s_cnt[own[kk]], 1);
    }
    __syncthreads();
    for (int j = threadIdx.x; j < cnt; j += kBlock)
      if (s_cnt[j] != 0) atomicAdd(&a.scnt[i0 + j], s_cnt[j]);
    __syncthreads();
  }
}

// Candidate order for the best prefix: smaller cut/den (exact), then smaller k.
__device__ __forceinline__ bool cand_better(long long oc, long long od, long long ok, long long xc,
                                            long long xd, long long xk) {
  if (ok <= 0) return false;
  if (xk <= 0) return true;
  if (ratio_lt(oc, od, xc, xd)) return true;
  return !ratio_lt(xc, xd, oc, od) && ok < xk;
}

__device__ void block_argmin(long long* s_bc, long long* s_bd, long long* s_bk) {
  for (int o = kBlock / 2; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) {
      const int u = threadIdx.x + o;
      if (cand_better(s_bc[u], s_bd[u], s_bk[u], s_bc[threadIdx.x], s_bd[threadIdx.x],
                      s_bk[threadIdx.x])) {
        s_bc[threadIdx.x] = s_bc[u];
        s_bd[threadIdx.x] = s_bd[u];
        s_bk[threadIdx.x] = s_bk[u];
      }
    }
    __syncthreads();
  }
}

// Reduce the per-block candidates of k_cut_scan (one workgroup; written by
// the others of the launch: device-scope reads).
__device__ void cut_final(const PlainArgs& a, Ctl* c, int N, long long* s_bc, long long* s_bd,
                          long long* s_bk) {
  const int nblk = (N + kScanBlock - 1) / kScanBlock;
  long long mc = -1, md = 1, mk = 0;
  for (int j = threadIdx.x; j < nblk; j += kBlock) {
    const long long jc = ld_agent(&a.bbest[3 * j]), jd = ld_agent(&a.bbest[3 * j + 1]),
                    jk = ld_agent(&a.bbest[3 * j + 2]);
    if (cand_better(jc, jd, jk, mc, md, mk)) { mc = jc; md = jd; mk = jk; }
  }
  s_bc[threadIdx.x] = mc; s_bd[threadIdx.x] = md; s_bk[threadIdx.x] = mk;
  __syncthreads();
  block_argmin(s_bc, s_bd, s_bk);
  if (threadIdx.x == 0) {
    long long bk = s_bk[0];
    c->kstar = bk > 0 ? bk : 0;
    c->best_cut = bk > 0 ? s_bc[0] : 0;
    c->best_den = bk > 0 ? s_bd[0] : 0;
    c->best_vol = bk > 0 ? a.svol[bk - 1] : 0;
    c->phi = bk > 0 ? (double)s_bc[0] / (double)s_bd[0] : 0.0;
  }
}

// Inclusive prefix of the boundary deltas gives |boundary(S_k)|; with vol_k
// the conductance of every prefix follows.  Each block publishes its best
// prefix (smallest cut/den by exact comparison, first k on ties, den = 0
// excluded), and resets p and the rank of its vertices, which no later step
// reads (r was reset by the block sort's side job).  The last workgroup
// reduces the candidates and marks the sweep finished.
__global__ __launch_bounds__(kBlock) void k_cut_scan(PlainArgs a) {
  Ctl* c = a.ctl;
  if (c->status != ST_SWEEPING) return;
  const int N = c->N;
  __shared__ long long sh[kBlock / 64 + 1];
  __shared__ long long s_excl;
  __shared__ unsigned long long s_tk;
  __shared__ int s_last;
  __shared__ long long s_bc[kBlock], s_bd[kBlock], s_bk[kBlock];
  const int nblk = (N + kScanBlock - 1) / kScanBlock;
  const bool fixed = scan_fixed(nblk);
  if (fixed && (int)blockIdx.x >= (nblk > 1 ? nblk : 1)) return;
  ScanSite* site = &c->scan[SCAN_CUT];
  unsigned long long* desc = nullptr;
  const long long vt = c->vol_total;
  int b = nblk;
  if (N > 0) b = scan_begin(site, a.desc[SCAN_CUT], a.desc_cap, nblk, fixed, &s_tk, &desc);
  for (; b < nblk; b = scan_next(site, nblk, fixed, &s_tk)) {
    // kScanItems consecutive positions per thread (see k_self)
    const int i0 = b * kScanBlock + (int)threadIdx.x * kScanItems;
    long long dk[kScanItems];
    long long dsum = 0;
#pragma unroll
    for (int k = 0; k < kScanItems; k++) {
      const int i = i0 + k;
      dk[k] = i < N ? (long long)a.sdeg[i] - 2ll * a.scnt[i] : 0;
      dsum += dk[k];
    }
#pragma unroll
    for (int k = 0; k < kScanItems; k++) {
      const int i = b * kScanBlock + k * kBlock + (int)threadIdx.x;
      if (i < N) {
        const int32_t v = a.sid[i];
        a.vr[v].rank = 0;
        a.p[v] = 0.0;
      }
    }
    long long agg;
    const long long ex = block_excl_scan<kBlock>(dsum, &agg, sh);
    if (threadIdx.x < 64) {
      const long long ex0 = scan_lookback(desc, b, agg, &c->fault);
      if (threadIdx.x == 0) s_excl = ex0;
    }
    __syncthreads();
    long long cut = s_excl + ex;
    long long mc = -1, md = 1, mk = 0;
#pragma unroll
    for (int k = 0; k < kScanItems; k++) {
      const int i = i0 + k;
      cut += dk[k];
      if (i < N) {
        const long long vol = a.svol[i];
        const long long den = vol < vt - vol ? vol : vt - vol;
        if (den > 0 && (mk <= 0 || ratio_lt(cut, den, mc, md))) { mc = cut; md = den; mk = i + 1; }
      }
    }
    s_bc[threadIdx.x] = mc; s_bd[threadIdx.x] = md; s_bk[threadIdx.x] = mk;
    __syncthreads();
    block_argmin(s_bc, s_bd, s_bk);
    if (threadIdx.x == 0) {
      // (exchanges that have returned are in place for the last workgroup)
      unsigned long long* bb = reinterpret_cast<unsigned long long*>(a.bbest) + 3 * (size_t)b;
      const unsigned long long o0 = atomicExch(&bb[0], (unsigned long long)s_bc[0]);
      const unsigned long long o1 = atomicExch(&bb[1], (unsigned long long)s_bd[0]);
      const unsigned long long o2 = atomicExch(&bb[2], (unsigned long long)s_bk[0]);
      asm volatile("" : : "v"(o0), "v"(o1), "v"(o2) : "memory");
    }
    __syncthreads();
  }
  const int members = !fixed ? (int)gridDim.x : nblk > 1 ? nblk : 1;
  if (members > 1 && !last_block_of(&c->done[DONE_FINISH], &s_last, false, (unsigned)members))
    return;
  if (N > 0) cut_final(a, c, N, s_bc, s_bd, s_bk);
  if (threadIdx.x == 0) {
    c->t_end = (long long)wall_clock64();
    c->status = ST_SWEPT;
  }
}

// ---------------------------------------------------------------- launchers

hipError_t launch_graph_init(hipStream_t s, const PlainArgs& a) {
  int grid = (int)((a.n + kBlock - 1) / kBlock);
  if (grid > 4096) grid = 4096;
  if (grid < 1) grid = 1;
  hipLaunchKernelGGL(k_graph_init, dim3(grid), dim3(kBlock), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_query_init(hipStream_t s, const PlainArgs& a, int32_t seed, int32_t rule,
                             double alpha, double eps, int32_t max_rounds, double beta) {
  hipLaunchKernelGGL(k_query_init, dim3(1), dim3(64), 0, s, a, seed, rule, alpha, eps,
                     max_rounds, beta);
  return hipGetLastError();
}

hipError_t launch_query_init_guarded(hipStream_t s, const PlainArgs& a, int32_t seed,
                                     int32_t rule, double alpha, double eps, int32_t max_rounds) {
  hipLaunchKernelGGL(k_query_init_guarded, dim3(1), dim3(64), 0, s, a, seed, rule, alpha, eps,
                     max_rounds);
  return hipGetLastError();
}

hipError_t launch_query_init_set(hipStream_t s, const PlainArgs& a, int32_t nseeds, int32_t rule,
                                 double alpha, double eps, int32_t max_rounds) {
  int grid = (nseeds + kBlock - 1) / kBlock;
  if (grid > 1024) grid = 1024;
  hipLaunchKernelGGL(k_query_init_set, dim3(grid), dim3(kBlock), 0, s, a, nseeds, rule, alpha, eps,
                     max_rounds);
  return hipGetLastError();
}

hipError_t launch_beta_pre(hipStream_t s, const PlainArgs& a, int grid, int64_t max_count) {
  hipLaunchKernelGGL(k_beta_keys, dim3(grid), dim3(kBlock), 0, s, a);
  SortArgs sa;
  sa.buf[0] = a.sbuf[0];
  sa.buf[1] = a.sbuf[1];
  sa.count = &a.ctl->N;
  sa.flip = &a.ctl->sort_flip;
  sa.active = nullptr;
  sa.active_value = 0;
  sa.rank = nullptr;
  hipError_t e = launch_sort(s, sa, max_count < a.n ? max_count : a.n, grid);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_beta_select, dim3(grid), dim3(kBlock), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_beta_post(hipStream_t s, const PlainArgs& a, int grid) {
  hipLaunchKernelGGL(k_beta_carry, dim3(grid), dim3(kBlock), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_hk_init(hipStream_t s, const PlainArgs& a, int32_t x, int32_t N, double t,
                          double A) {
  hipLaunchKernelGGL(k_hk_init, dim3(1), dim3(64), 0, s, a, x, N, t, A);
  return hipGetLastError();
}

hipError_t launch_hk_level(hipStream_t s, const PlainArgs& a, int grid_self, int grid_scatter) {
  hipLaunchKernelGGL(k_hk_self, dim3(grid_self), dim3(kBlock), 0, s, a);
  hipLaunchKernelGGL(k_hk_scatter, dim3(grid_scatter), dim3(kBlock), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_nb_init(hipStream_t s, const PlainArgs& a, int32_t x, double eps, int32_t T) {
  hipLaunchKernelGGL(k_nb_init, dim3(1), dim3(64), 0, s, a, x, eps, T);
  return hipGetLastError();
}

hipError_t launch_nb_step(hipStream_t s, const PlainArgs& a, int grid_self, int grid_scatter,
                          int grid_bin) {
  hipLaunchKernelGGL(k_nb_self, dim3(grid_self), dim3(kBlock), 0, s, a);
  hipLaunchKernelGGL(k_nb_scatter, dim3(grid_scatter), dim3(kBlock), 0, s, a, (int)(grid_bin > 0));
  if (grid_bin > 0)
    hipLaunchKernelGGL(k_bin_apply<kModeNB>, dim3(grid_bin), dim3(kBlock), 0, s, a, -1);
  return hipGetLastError();
}

hipError_t launch_nb_finish(hipStream_t s, const PlainArgs& a, int32_t R, int32_t J, int grid) {
  hipLaunchKernelGGL(k_nb_finish, dim3(grid), dim3(kBlock), 0, s, a, R, J);
  return hipGetLastError();
}

hipError_t launch_hk_clear(hipStream_t s, const PlainArgs& a, int grid) {
  hipLaunchKernelGGL(k_hk_clear, dim3(grid), dim3(kBlock), 0, s, a);
  return hipGetLastError();
}

// At most one workgroup per block of rows, at most 2048 (the whole chip).
static int dense_grid(const PlainArgs& a) {
  constexpr int most = kDenseGroup * kDenseGroups;
  return a.ndblk < most ? a.ndblk : most;
}

hipError_t launch_dense(hipStream_t s, const PlainArgs& a, hipEvent_t t0, hipEvent_t t1,
                        int slot) {
  if (slot >= kMaxChunk || a.ndblk < 1) return hipErrorInvalidValue;
  if (t0)
    hipExtLaunchKernelGGL(k_dense, dim3(dense_grid(a)), dim3(kBlock), 0, s, t0, t1, 0, a, slot);
  else
    hipLaunchKernelGGL(k_dense, dim3(dense_grid(a)), dim3(kBlock), 0, s, a, slot);
  return hipGetLastError();
}

hipError_t launch_light_self(hipStream_t s, const PlainArgs& a, int grid, hipEvent_t t0,
                             hipEvent_t t1, int slot) {
  if (slot >= kMaxChunk) return hipErrorInvalidValue;
  if (t0)
    hipExtLaunchKernelGGL(k_light_self, dim3(grid), dim3(kBlock), 0, s, t0, t1, 0, a, slot);
  else
    hipLaunchKernelGGL(k_light_self, dim3(grid), dim3(kBlock), 0, s, a, slot);
  return hipGetLastError();
}

hipError_t launch_hk_light(hipStream_t s, const PlainArgs& a, int grid_self, int grid_scatter) {
  hipLaunchKernelGGL(k_hk_light_self, dim3(grid_self), dim3(kBlock), 0, s, a);
  hipLaunchKernelGGL(k_hk_scatter, dim3(grid_scatter), dim3(kBlock), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_hk_dense(hipStream_t s, const PlainArgs& a) {
  if (a.ndblk < 1) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_hk_dense, dim3(dense_grid(a)), dim3(kBlock), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_self(hipStream_t s, const PlainArgs& a, int grid, hipEvent_t t0, hipEvent_t t1,
                       int slot) {
  if (slot >= kMaxChunk) return hipErrorInvalidValue;
  if (t0)
    hipExtLaunchKernelGGL(k_self, dim3(grid), dim3(kSelfBlk), 0, s, t0, t1, 0, a, slot);
  else
    hipLaunchKernelGGL(k_self, dim3(grid), dim3(kSelfBlk), 0, s, a, slot);
  return hipGetLastError();
}

hipError_t launch_scatter(hipStream_t s, const PlainArgs& a, int grid, hipEvent_t t0,
                          hipEvent_t t1, int slot, int grid_bin, int pair, bool apply_wanted) {
  if (slot >= kMaxChunk || pair >= 32) return hipErrorInvalidValue;
  // k_bin_apply only where a round can be binned (an empty
  // launch still costs a dispatch every round)
  const bool apply = apply_wanted && bins_possible(a);
  const int ap = apply ? 1 : 0;
  if (t0) {
    hipExtLaunchKernelGGL(k_scatter, dim3(grid), dim3(kBlock), 0, s, t0, apply ? nullptr : t1, 0,
                          a, slot, pair, ap);
    if (apply)
      hipExtLaunchKernelGGL(k_bin_apply<kModePR>, dim3(grid_bin), dim3(kBlock), 0, s, nullptr, t1, 0, a,
                            slot);
  } else {
    hipLaunchKernelGGL(k_scatter, dim3(grid), dim3(kBlock), 0, s, a, slot, pair, ap);
    if (apply) hipLaunchKernelGGL(k_bin_apply<kModePR>, dim3(grid_bin), dim3(kBlock), 0, s, a, slot);
  }
  return hipGetLastError();
}

// A finished query's results, from the sweep's buffers into its result
// block: the support in sweep order with p, and the nonzeros of r.
__global__ __launch_bounds__(kBlock) void k_copy_result(PlainArgs a, int32_t* ids, double* p,
                                                        int32_t* rid, double* rval, int N, int R) {
  const int stride = gridDim.x * kBlock;
  for (int i = blockIdx.x * kBlock + threadIdx.x; i < N; i += stride) {
    ids[i] = a.sid[i];
    p[i] = a.sp[i];
  }
  for (int i = blockIdx.x * kBlock + threadIdx.x; i < R; i += stride) {
    rid[i] = a.rid[i];
    rval[i] = a.rval[i];
  }
}

hipError_t launch_copy_result(hipStream_t s, const PlainArgs& a, int32_t* ids, double* p,
                              int32_t* rid, double* rval, int N, int R, int grid) {
  if (N < 0 || R < 0 || N > a.n || R > a.n) return hipErrorInvalidValue;
  if (N == 0 && R == 0) return hipSuccess;
  hipLaunchKernelGGL(k_copy_result, dim3(grid), dim3(kBlock), 0, s, a, ids, p, rid, rval, N, R);
  return hipGetLastError();
}

// Before the read-back that tells the sizes, so that a query ends with it: one
// query on R-MAT 2^12 takes 144 us (163 with the copy launched after it, another
// launch and wait), on R-MAT 2^20 268 (288).
__global__ __launch_bounds__(kBlock) void k_copy_ahead(PlainArgs a, char* block,
                                                       unsigned long long cap, int residual) {
  Ctl* c = a.ctl;
  const long long N = c->N, R = residual ? c->rnnz : 0;
  bool go = c->status == ST_SWEPT && !c->fault && N >= 0 && N <= a.n && R >= 0 && R <= a.n;
  const ResultLayout l = result_layout(go ? (size_t)N : 0, go ? (size_t)R : 0);
  go = go && l.bytes <= cap;
  if (blockIdx.x == 0 && threadIdx.x == 0) c->copied = go;
  if (!go) return;
  int32_t* ids = reinterpret_cast<int32_t*>(block);
  double* p = reinterpret_cast<double*>(block + l.p);
  int32_t* rid = reinterpret_cast<int32_t*>(block + l.rid);
  double* rval = reinterpret_cast<double*>(block + l.rval);
  const long long stride = (long long)gridDim.x * kBlock;
  for (long long i = (long long)blockIdx.x * kBlock + threadIdx.x; i < N; i += stride) {
    ids[i] = a.sid[i];
    p[i] = a.sp[i];
  }
  for (long long i = (long long)blockIdx.x * kBlock + threadIdx.x; i < R; i += stride) {
    rid[i] = a.rid[i];
    rval[i] = a.rval[i];
  }
}

hipError_t launch_copy_ahead(hipStream_t s, const PlainArgs& a, void* block, size_t cap,
                             bool residual, int grid) {
  hipLaunchKernelGGL(k_copy_ahead, dim3(grid), dim3(kBlock), 0, s, a, static_cast<char*>(block),
                     (unsigned long long)cap, (int)residual);
  return hipGetLastError();
}

// Several results' parts into one destination (the host's pinned staging
// memory): one workgroup per part at a time, 16-byte words where both ends
// allow it.
__global__ __launch_bounds__(kBlock) void k_gather_results(const GatherJob* jobs, int njobs,
                                                           uint32_t* dst) {
  for (int j = blockIdx.x; j < njobs; j += gridDim.x) {
    const GatherJob J = jobs[j];
    const uint32_t* src = J.src;
    uint32_t* out = dst + J.dst_off;
    const uint64_t nw = J.words;
    const bool wide = ((reinterpret_cast<uintptr_t>(src) | reinterpret_cast<uintptr_t>(out)) & 15) == 0;
    const uint64_t n4 = wide ? nw / 4 : 0;
    for (uint64_t i = threadIdx.x; i < n4; i += kBlock)
      reinterpret_cast<uint4*>(out)[i] = reinterpret_cast<const uint4*>(src)[i];
    for (uint64_t i = 4 * n4 + threadIdx.x; i < nw; i += kBlock) out[i] = src[i];
  }
}

hipError_t launch_gather_results(hipStream_t s, const GatherJob* jobs, int njobs, uint32_t* dst) {
  if (njobs <= 0) return hipSuccess;
  const int grid = njobs < 1024 ? njobs : 1024;
  hipLaunchKernelGGL(k_gather_results, dim3(grid), dim3(kBlock), 0, s, jobs, njobs, dst);
  return hipGetLastError();
}

hipError_t launch_sweep(hipStream_t s, const PlainArgs& a, int grid, int64_t max_count) {
  hipLaunchKernelGGL(k_sweep_keys, dim3(grid), dim3(kBlock), 0, s, a, (long long)max_count);
  SortArgs sa;
  sa.buf[0] = a.sbuf[0];
  sa.buf[1] = a.sbuf[1];
  sa.count = &a.ctl->N;
  sa.flip = &a.ctl->sort_flip;
  sa.active = &a.ctl->status;
  sa.active_value = ST_SWEEPING;
  // the volume prefix is written only after the sort: its words hold the
  // small-count path's rank accumulators meanwhile
  sa.rank = reinterpret_cast<unsigned long long*>(a.svol);
  // the block sort's workgroups without a tile gather the nonzeros of r over
  // the touched list into the result buffers and reset r (no later sweep
  // kernel reads r)
  static_assert(sizeof(VRec) % sizeof(double) == 0, "r read with a stride of whole records");
  sa.side_ids = a.touched;
  sa.side_count = &a.ctl->touched_cnt;
  sa.side_val = &a.vr[0].r;
  sa.side_stride = (int)(sizeof(VRec) / sizeof(double));
  sa.side_out_id = a.rid;
  sa.side_out_val = a.rval;
  sa.side_out_cnt = &a.ctl->rnnz;
  sa.side_out_cap = a.n;
  sa.side_fault = &a.ctl->fault;
  hipError_t e = launch_sort(s, sa, max_count < a.n ? max_count : a.n, grid);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_vol_scan, dim3(grid), dim3(kBlock), 0, s, a);
  // the count walks many short, latency-bound steps: a larger grid keeps
  // each workgroup to about one
  hipLaunchKernelGGL(k_cut_count, dim3(4 * grid), dim3(kBlock), 0, s, a);
  hipLaunchKernelGGL(k_cut_scan, dim3(grid), dim3(kBlock), 0, s, a);
  return hipGetLastError();
}

}  // namespace plc
