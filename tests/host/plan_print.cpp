// Prints the work decomposition of FFT searches, one line "<ranges> <items>" per line
// "<bins> <templates per bin> <L> <blocks of offsets> <CUs> <tails> <t_block>" on stdin (tails: 1
// for a tail search).  With the argument "tiles", the tile of FP32 searches, "<template blocks>
// <offset blocks> <offsets per work item>" per line "<bins> <templates per bin> <L> <offsets>
// <CUs>"; with "cuts", an FFT search's ranges that cut bins, 0 for whole bins, per line "<bins>
// <templates per bin> <L> <offsets> <CUs>" (one series).
// Host code only: the planner needs no device.  Exit status 2 if bf_plan
// does not refuse a series shorter than L by its length, GPU or none.
#include "bfly_runtime.h"

#include <cstdio>

static void print_cuts() {
  int n_bins, n_fdot, L, slots;
  long long W;
  while (std::scanf("%d %d %d %lld %d", &n_bins, &n_fdot, &L, &W, &slots) == 5) {
    bfly::BankDev b = {};
    b.precision = bfly::P_FFT;
    b.fft_m = 4096;
    b.L = L;
    b.n_bins = n_bins;
    b.n_fdot = n_fdot;
    b.K = (int64_t)n_bins * n_fdot;
    bfly::SearchDev sp = {};
    sp.t_block = 1;
    const int64_t blocks = bfly::fft_blocks(b, W);
    const int32_t whole = bfly::plan_fft_ranges(b, blocks, slots, sp);
    std::printf("%d\n", bfly::plan_split_ranges(b, blocks, W, slots, whole));
  }
}

static void print_tiles() {
  int n_bins, n_fdot, L, slots;
  long long W;
  while (std::scanf("%d %d %d %lld %d", &n_bins, &n_fdot, &L, &W, &slots) == 5) {
    bfly::BankDev b = {};
    b.precision = bfly::P_FP32;
    b.L = L;
    b.n_bins = n_bins;
    b.n_fdot = n_fdot;
    b.K = (int64_t)n_bins * n_fdot;
    b.L_pad = (L + 31) / 32 * 32;
    const bf_search_params prm = {BF_NORM_CENTRED, 1, 1, 0, 0.0, 1.0};
    bfly::SearchDev sp = bfly::make_search(b, &prm);
    bf_segment seg = {};
    seg.n = W + L - 1;
    bfly::fit_tile(b, &seg, 1, slots, &sp);
    std::printf("%d %d %d\n", sp.tm, sp.tn, sp.n_wg);
  }
}

int main(int argc, char** argv) {
  bf_bank bank = {};
  bank.dev.L = 64;
  const int64_t n[2] = {64, 63};
  if (bf_plan(&bank, n, 2, nullptr, nullptr) != BF_EINVAL) return 2;
  if (argc > 1) {
    argv[1][0] == 't' ? print_tiles() : print_cuts();
    return 0;
  }
  int n_bins, n_fdot, L, slots, tails, t_block;
  long long blocks;
  while (std::scanf("%d %d %d %lld %d %d %d", &n_bins, &n_fdot, &L, &blocks, &slots, &tails,
                    &t_block) == 7) {
    bfly::BankDev b = {};
    b.precision = bfly::P_FFT;
    b.fft_m = 4096;
    b.L = L;
    b.n_bins = n_bins;
    b.n_fdot = n_fdot;
    b.K = (int64_t)n_bins * n_fdot;
    bfly::SearchDev sp = {};
    sp.mode = tails ? bfly::MODE_ONEPASS : bfly::MODE_SEARCH;
    sp.t_block = t_block;
    const int32_t r = bfly::plan_fft_ranges(b, blocks, slots, sp);
    std::printf("%d %lld\n", r, blocks * r);
  }
  return 0;
}
