// device_util.h -- wavefront / workgroup building blocks shared by the
// libplc kernels (CDNA, 64-lane wavefronts, 256-thread workgroups).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "scan_site.h"

namespace plc {

#define PLC_LANE (threadIdx.x & 63)
#define PLC_WID (threadIdx.x >> 6)

__device__ __forceinline__ unsigned long long lanemask_lt() {
  unsigned l = PLC_LANE;
  return l == 0 ? 0ull : (~0ull >> (64 - l));
}

__device__ __forceinline__ long long wave_incl_scan(long long x) {
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    long long y = __shfl_up(x, o);
    if ((int)PLC_LANE >= o) x += y;
  }
  return x;
}

// Exclusive scan over a workgroup of NT threads; sh holds NT/64 + 1 slots.
template <int NT>
__device__ __forceinline__ long long block_excl_scan(long long x, long long* total, long long* sh) {
  constexpr int NW = NT / 64;
  long long inc = wave_incl_scan(x);
  if (PLC_LANE == 63) sh[PLC_WID] = inc;
  __syncthreads();
  if (threadIdx.x < 64) {
    long long v = (int)threadIdx.x < NW ? sh[threadIdx.x] : 0;
    long long vi = wave_incl_scan(v);
    if ((int)threadIdx.x < NW) sh[threadIdx.x] = vi - v;
    if ((int)threadIdx.x == NW - 1) sh[NW] = vi;
  }
  __syncthreads();
  long long ex = inc - x + sh[PLC_WID];
  *total = sh[NW];
  __syncthreads();
  return ex;
}

// ----------------------------------------------------------- look-back scan
//
// Single-pass (decoupled look-back) scan over blocks taken in ticket order.
// One 64-bit word per block holds the flag (bits 63..62: 0 none,
// 1 aggregate, 2 inclusive prefix) and a 62-bit two's-complement value, so a
// reader never needs a memory fence between flag and value.  Each scan site
// owns two descriptor buffers used on alternate launches; every launch clears
// the slots the previous launch used in the other buffer, so the next launch
// starts from zeroed flags.

__device__ __forceinline__ unsigned long long desc_pack(unsigned flag, long long v) {
  return ((unsigned long long)flag << 62) | ((unsigned long long)v & ((1ull << 62) - 1));
}
__device__ __forceinline__ long long desc_value(unsigned long long w) {
  return ((long long)(w << 2)) >> 2;
}
__device__ __forceinline__ unsigned long long atomic_ld64(unsigned long long* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void atomic_st64(unsigned long long* p, unsigned long long v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

constexpr long kSpinLimit = 1L << 24;

// Scans of few blocks: the first nblk workgroups draw one ticket each and those
// past them leave at once, so that the site's word, to which every workgroup of
// the launch adds otherwise (~10 ns each, one after another), gets nblk
// additions only.  The block a workgroup takes is its ticket and not its own
// number: workgroups start in no order across XCDs, and where another stream's
// launches hold part of the chip, one that waited for a lower number could
// keep out of its place the very workgroup it waits for.  The holder of a lower
// ticket has started.  kScanFixed: at most so many such additions, a block per
// CU.
constexpr int kScanFixed = 256;
__device__ __forceinline__ bool scan_fixed(int nblk) {
  return nblk <= kScanFixed && nblk <= (int)gridDim.x;
}

// A draw (one thread): the site's word before it.  The last draw of the launch
// leaves the word of the next one.
__device__ __forceinline__ unsigned long long scan_draw(ScanSite* site, int nblk, bool fixed) {
  const unsigned long long w = atomicAdd(&site->word, 1ull);
  if (scan_ticket_of(w) == scan_draws(nblk, (int)gridDim.x, fixed) - 1)
    atomic_st64(&site->word, scan_after(w, nblk));
  return w;
}

// The workgroup's first block (>= nblk: none) and the launch's descriptors.
// With fixed only the first nblk workgroups call it, and one alone draws
// nothing: it has no descriptors, and the site stays as it was.  sh: one LDS
// word, which scan_next takes too.
__device__ __forceinline__ int scan_begin(ScanSite* site, unsigned long long* desc2, int cap,
                                          int nblk, bool fixed, unsigned long long* sh,
                                          unsigned long long** desc) {
  *desc = nullptr;
  if (fixed && nblk == 1) {
    __syncthreads();
    return 0;
  }
  if (threadIdx.x == 0) *sh = scan_draw(site, nblk, fixed);
  __syncthreads();
  const unsigned long long w = *sh;
  const unsigned par = scan_parity_of(w);
  *desc = desc2 + (size_t)par * cap;
  // the slots of the previous launch, shared out among the workgroups here
  unsigned long long* const other = desc2 + (size_t)(par ^ 1u) * cap;
  const int prev = scan_prev_of(w) < cap ? scan_prev_of(w) : cap;
  const int m = fixed ? nblk : (int)gridDim.x;
  for (int j = blockIdx.x * blockDim.x + threadIdx.x; j < prev; j += m * blockDim.x)
    other[j] = 0ull;
  return scan_ticket_of(w);
}
// The workgroup's next block (>= nblk: none).
__device__ __forceinline__ int scan_next(ScanSite* site, int nblk, bool fixed,
                                         unsigned long long* sh) {
  if (fixed) return nblk;
  __syncthreads();
  if (threadIdx.x == 0) *sh = scan_draw(site, nblk, fixed);
  __syncthreads();
  return scan_ticket_of(*sh);
}

// Decoupled look-back for block b, by the 64 lanes of wave 0 together (call
// from threads 0..63; every lane gets the result).  Each round reads the
// descriptors of the 64 nearest unresolved predecessors at once and sums
// back to the nearest inclusive prefix; lanes past block 0 count as an
// inclusive prefix of 0.  A round that meets a predecessor without a
// descriptor before any inclusive one waits and reads again.  Predecessors
// drew their tickets earlier, so they are running or done; the wait is
// bounded and raises *fault if it ever runs out.  Returns the exclusive
// prefix.  desc: null where there is one block only.
__device__ long long scan_lookback(unsigned long long* desc, int b, long long agg, int* fault) {
  const int lane = PLC_LANE;
  if (b == 0) {
    if (lane == 0 && desc) atomic_st64(&desc[0], desc_pack(2, agg));
    return 0;
  }
  if (lane == 0) atomic_st64(&desc[b], desc_pack(1, agg));
  long long excl = 0;
  int j = b - 1;  // nearest predecessor not yet summed
  long spins = 0;
  for (;;) {
    const int idx = j - lane;
    const unsigned long long w = idx >= 0 ? atomic_ld64(&desc[idx]) : desc_pack(2, 0);
    const unsigned flag = (unsigned)(w >> 62);
    const unsigned long long incl = __ballot(flag == 2);
    const unsigned long long none = __ballot(flag == 0);
    const int fi = incl ? __ffsll((long long)incl) - 1 : 64;
    const int fz = none ? __ffsll((long long)none) - 1 : 64;
    if (fz < fi) {
      if (++spins > kSpinLimit) {
        if (lane == 0) atomicExch(fault, 1);
        break;
      }
      __builtin_amdgcn_s_sleep(1);
      continue;
    }
    long long v = lane <= fi ? desc_value(w) : 0;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    excl += v;
    if (fi < 64) break;
    j -= 64;
  }
  if (lane == 0) atomic_st64(&desc[b], desc_pack(2, excl + agg));
  return excl;
}

// Last-workgroup detection: true in exactly one workgroup, after all others
// of the launch called it.  with_acquire makes the other workgroups' global
// writes visible to the last one (device-scope fences).
// last_block_of: the same among the first `members` workgroups only (the
// others must not call it).
__device__ __forceinline__ bool last_block_of(unsigned* done, int* sh, bool with_acquire,
                                              unsigned members) {
  __syncthreads();
  if (threadIdx.x == 0) {
    if (with_acquire) __threadfence();
    unsigned prev = atomicAdd(done, 1u);
    int last = prev == members - 1;
    if (last) {
      if (with_acquire) __threadfence();
      *done = 0;
    }
    *sh = last;
  }
  __syncthreads();
  int l = *sh;
  __syncthreads();
  return l != 0;
}

__device__ __forceinline__ bool last_block(unsigned* done, int* sh, bool with_acquire) {
  __syncthreads();
  if (threadIdx.x == 0) {
    if (with_acquire) __threadfence();
    unsigned prev = atomicAdd(done, 1u);
    int last = prev == gridDim.x - 1;
    if (last) {
      if (with_acquire) __threadfence();
      *done = 0;
    }
    *sh = last;
  }
  __syncthreads();
  int l = *sh;
  __syncthreads();
  return l != 0;
}

// Wavefront-ballot append into an LDS staging buffer: the lanes of the
// calling wave with pred set store v at consecutive slots of buf, reserved
// with one LDS atomic per wave (the popcount of the ballot); a lane's slot
// is the number of set lanes below it.  Safe in divergent code: only the
// active lanes take part.
__device__ __forceinline__ void wave_append(bool pred, int32_t v, int32_t* buf, int* cnt) {
  const unsigned long long m = __ballot(pred);
  if (m == 0ull) return;
  const int leader = __ffsll((long long)m) - 1;
  int base = 0;
  if ((int)PLC_LANE == leader) base = atomicAdd(cnt, __popcll(m));
  base = __shfl(base, leader);
  if (pred) buf[base + __popcll(m & lanemask_lt())] = v;
}

// The same for up to K values per lane, those of the bits set in pred: one
// LDS atomic per wave for all of them (each is a round trip to LDS, one after
// another otherwise).
template <int K>
__device__ __forceinline__ void wave_append_all(unsigned pred, const int32_t (&v)[K],
                                                int32_t* buf, int* cnt) {
  int n = __popc(pred);  // inclusive scan of the lanes' counts
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int y = __shfl_up(n, o);
    if ((int)PLC_LANE >= o) n += y;
  }
  const int tot = __shfl(n, 63);
  if (tot == 0) return;
  int base = 0;
  if (PLC_LANE == 63) base = atomicAdd(cnt, tot);
  int at = __shfl(base, 63) + n - __popc(pred);
#pragma unroll
  for (int k = 0; k < K; k++)
    if ((pred >> k) & 1u) buf[at++] = v[k];
}

// Workgroup-aggregated append of the values staged in an LDS buffer:
// one global atomic per call.  Every thread must call it.  Writes
// dst[base + j] = buf[j] for j < *count (slots >= cap raise *fault).
__device__ __forceinline__ void block_flush(int32_t* counter, int32_t* dst, int64_t cap,
                                            const int32_t* buf, int* count, int* s_base,
                                            int* fault) {
  __syncthreads();
  int cnt = *count;
  if (threadIdx.x == 0) *s_base = cnt > 0 ? atomicAdd(counter, cnt) : 0;
  __syncthreads();
  long long base = *s_base;
  for (int j = threadIdx.x; j < cnt; j += blockDim.x) {
    long long slot = base + j;
    if (slot < cap) dst[slot] = buf[j]; else *fault = 1;
  }
  __syncthreads();
  if (threadIdx.x == 0) *count = 0;
  __syncthreads();
}

// Two lists at once (block_flush for each): the two reservations are in
// flight together and share the barriers.
__device__ __forceinline__ void block_flush2(int32_t* ctr0, int32_t* dst0, const int32_t* buf0,
                                             int* cnt0, int32_t* ctr1, int32_t* dst1,
                                             const int32_t* buf1, int* cnt1, int64_t cap,
                                             int* s_base /* 2 */, int* fault) {
  __syncthreads();
  const int n0 = *cnt0, n1 = *cnt1;
  if (threadIdx.x < 2) {
    const int m = threadIdx.x == 0 ? n0 : n1;
    s_base[threadIdx.x] = m > 0 ? atomicAdd(threadIdx.x == 0 ? ctr0 : ctr1, m) : 0;
  }
  __syncthreads();
  const long long b0 = s_base[0], b1 = s_base[1];
  for (int j = threadIdx.x; j < n0; j += blockDim.x) {
    if (b0 + j < cap) dst0[b0 + j] = buf0[j]; else *fault = 1;
  }
  for (int j = threadIdx.x; j < n1; j += blockDim.x) {
    if (b1 + j < cap) dst1[b1 + j] = buf1[j]; else *fault = 1;
  }
  if (threadIdx.x == 0) {
    *cnt0 = 0;
    *cnt1 = 0;
  }
  __syncthreads();
}

// The dispatcher hands workgroups to the 8 XCDs round-robin (XCD =
// blockIdx % 8), and each XCD has its own L2.  xcd_block renumbers the
// workgroups of a grid of G so that those of one XCD get consecutive numbers
// (a bijection on [0, G)).  A kernel that gives contiguous work ranges by
// this number keeps neighbouring work -- in the batched kernels, the edges of
// one slot, whose state lines they share -- inside one L2.
__device__ __forceinline__ int xcd_block(int b, int G) {
  const int q = G >> 3, r = G & 7, x = b & 7, i = b >> 3;
  return x * q + (x < r ? x : r) + i;
}

// a/b < c/d exactly, for b, d > 0.
__device__ __forceinline__ bool ratio_lt(long long a, long long b, long long c, long long d) {
  return (__int128)a * (__int128)d < (__int128)c * (__int128)b;
}

}  // namespace plc
