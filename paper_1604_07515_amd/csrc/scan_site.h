// scan_site.h -- the word through which the workgroups of a look-back scan
// share out its blocks (see device_util.h).
#pragma once
#include <hip/hip_runtime.h>

namespace plc {

// Bits 31..0: tickets drawn in this launch.  Bit 32: which of the site's two
// descriptor buffers the launch uses.  Bits 63..33: blocks of the launch
// before it, whose descriptors (in the other buffer) this one clears.  One
// atomic addition of 1 draws a ticket and tells the rest.
struct ScanSite {
  unsigned long long word, pad;
};

__host__ __device__ inline int scan_ticket_of(unsigned long long w) {
  return (int)(w & 0xffffffffull);
}
__host__ __device__ inline unsigned scan_parity_of(unsigned long long w) {
  return (unsigned)(w >> 32) & 1u;
}
__host__ __device__ inline int scan_prev_of(unsigned long long w) { return (int)(w >> 33); }

// Draws of a launch: the first nblk workgroups one each (and the others none),
// or every workgroup until it gets no block.
__host__ __device__ inline int scan_draws(int nblk, int grid, bool one_each) {
  return one_each ? nblk : nblk + grid;
}
// The word that the last draw (w, of nblk blocks) leaves for the next launch.
__host__ __device__ inline unsigned long long scan_after(unsigned long long w, int nblk) {
  return (unsigned long long)(unsigned)nblk << 33 |
         (unsigned long long)(scan_parity_of(w) ^ 1u) << 32;
}

}  // namespace plc
