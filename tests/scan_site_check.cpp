// The block shares of a look-back scan (scan_site.h), on the CPU.
// 1. Over launches of every kind the word hands out each block once, and tells
//    the descriptor buffer and the previous launch's blocks.
// 2. Three launches on different streams share a chip of 4 XCDs with two places
//    each, which fill them in any order: a workgroup keeps its place until
//    every lower block's workgroup has started.  With the block drawn as a
//    ticket every schedule ends; with the workgroup's own number as its block
//    some do not.
// Built and run by test_scan_site.py.
#include <cstdio>
#include <random>
#include <vector>

#include "../paper_1604_07515_amd/csrc/scan_site.h"

#define CHECK(c)                                                        \
  do {                                                                  \
    if (!(c)) {                                                         \
      std::fprintf(stderr, "check failed line %d: %s\n", __LINE__, #c); \
      return 1;                                                         \
    }                                                                   \
  } while (0)

static unsigned long long draw(plc::ScanSite& s, int nblk, int grid, bool one_each) {
  const unsigned long long w = s.word++;
  if (plc::scan_ticket_of(w) == plc::scan_draws(nblk, grid, one_each) - 1)
    s.word = plc::scan_after(w, nblk);
  return w;
}

constexpr int kXcd = 4, kPlaces = 2, kLaunches = 3, kBlk = 8, kGrid = 11;

// One schedule; false if it gets stuck.
static bool schedule(std::mt19937& rng, bool tickets) {
  plc::ScanSite site[kLaunches] = {};
  int started[kLaunches][kXcd] = {};          // workgroups of the launch started per XCD
  std::vector<char> on[kLaunches];            // block: its workgroup has started
  struct Wg { int launch, block; };
  std::vector<Wg> at[kXcd];
  for (auto& o : on) o.assign(kBlk, 0);
  for (;;) {
    // leave: idle workgroups at once, the others when every lower block is on
    for (auto& x : at)
      for (size_t i = 0; i < x.size();) {
        bool free = true;
        for (int b = 0; b < x[i].block && b < kBlk; b++) free &= on[x[i].launch][b] != 0;
        if (x[i].block >= kBlk || free) x.erase(x.begin() + (long)i); else i++;
      }
    // start one more workgroup: any XCD with a place, any launch with one left there
    std::vector<int> can;
    bool left = false;
    for (int x = 0; x < kXcd; x++)
      for (int l = 0; l < kLaunches; l++) {
        const int w = x + kXcd * started[l][x];
        if (w >= kGrid) continue;
        left = true;
        if ((int)at[x].size() < kPlaces) can.push_back(x * kLaunches + l);
      }
    if (can.empty()) return !left;
    const int pick = can[rng() % can.size()], x = pick / kLaunches, l = pick % kLaunches;
    const int w = x + kXcd * started[l][x]++;
    int b = kBlk;  // none
    if (w < kBlk) b = tickets ? plc::scan_ticket_of(draw(site[l], kBlk, kGrid, true)) : w;
    if (b < kBlk) on[l][b] = 1;
    at[x].push_back(Wg{l, b});
  }
}

int main() {
  std::mt19937 rng(7);
  plc::ScanSite s{};
  unsigned parity = 0;
  int prev = 0;
  for (int it = 0; it < 2000; it++) {
    const bool one_each = rng() & 1;
    const int grid = 1 + (int)(rng() % 600);
    const int nblk = 1 + (int)(rng() % (one_each ? (unsigned)grid : 3000u));
    const int draws = plc::scan_draws(nblk, grid, one_each);
    for (int k = 0; k < draws; k++) {
      const unsigned long long w = draw(s, nblk, grid, one_each);
      CHECK(plc::scan_ticket_of(w) == k && plc::scan_parity_of(w) == parity &&
            plc::scan_prev_of(w) == prev);
    }
    parity ^= 1;
    prev = nblk;
  }
  int stuck = 0;
  for (int it = 0; it < 20000; it++) {
    CHECK(schedule(rng, true));
    stuck += !schedule(rng, false);
  }
  CHECK(stuck > 0);
  std::printf("scan ok (%d of 20000 schedules stuck with fixed numbers)\n", stuck);
  return 0;
}
