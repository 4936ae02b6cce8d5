// Order of the 128 x 128 tiles of the sliced pair products (pair_bf16_v.hip, pair_i8_v.hip).
#pragma once
#include <hip/hip_runtime.h>

namespace dfpt2 {

// Workgroups are dealt round-robin to the 8 XCDs; each XCD gets a contiguous range of
// (pair, tile).  Tiles of one pair go in bands of 6 tile rows, column by column within a
// band: the ~32 workgroups resident on one XCD then read about 6 + 5 panels instead of the
// 14 of 3-4 whole tile rows (1% faster than row order).  Tiles with at most half their columns
// or rows, which take half as long, come after the whole tiles of all pairs.  31 holes, 539
// virtuals, BF16: product 4.30 -> 4.22 ms; workgroups of equal length stay at the same chunks of the
// panels that they share and find them in the L2 (57 -> 29% of the requests miss).  80 holes, 1200
// virtuals, 4000 auxiliary functions: 47.4 -> 46.2 ms per launch, though the misses rise there (24 -> 31% of
// the requests: strips of half tiles share fewer panels); what the gain comes from is not shown.
__device__ inline void v_tile(int h0, int n_v, int n_pairs, int& p, int& I, int& J) {
  constexpr int TV = 128, HB = 6;
  auto xcd = [](int h, int nblk) {
    const int x = h & 7, k = h >> 3, q = nblk >> 3, rem = nblk & 7;
    return (x < rem) ? x * (q + 1) + k : rem * (q + 1) + (x - rem) * q + k;
  };
  const int nt = (n_v + TV - 1) / TV, edge = n_v - (nt - 1) * TV;
  const int nf = edge <= TV / 2 ? nt - 1 : nt;  // whole tiles along either index
  const int full = nf * nf, rest = nt * nt - full, all = full * n_pairs;
  if (h0 < all) {
    const int L = xcd(h0, all);
    p = L / full;
    const int t = L - p * full, band = t / (HB * nf), h = min(HB, nf - band * HB), r = t - band * HB * nf;
    J = r / h;
    I = band * HB + (r - J * h);
  } else {  // the last column, then the last row
    const int L = xcd(h0 - all, rest * n_pairs);
    p = L / rest;
    const int t = L - p * rest;
    I = min(t, nf);
    J = t < nf ? nf : t - nf;
  }
}

}  // namespace dfpt2
