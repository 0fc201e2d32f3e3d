// The hop kernel that spreads the eight hops of a site over a workgroup (split.hip), and the
// 32-bit site arithmetic it shares with the gauge kernels.
#pragma once
#include "internal.h"

namespace sap {

// division of 0 <= n < 2^31 by a divisor known at launch: floor(n / d) = (n * m) >> s with
// s = 31 + ceil(log2 d), m = floor(2^s / d) + 1
struct FastDiv {
  unsigned m;
  int s;
};
inline FastDiv fast_div(int d) {
  FastDiv f;
  int l = 0;
  while ((1LL << l) < d) ++l;
  f.s = 31 + l;
  f.m = (unsigned)((1ULL << f.s) / (unsigned)d + 1);
  return f;
}
// the divisors of the site decomposition (a parity has fewer than 2^31 sites: its links
// alone take 1.1 KB a site)
struct SiteDiv {
  FastDiv d3, d2, d1, dv;   // L3 / 2, L2, L1, V3h
};
inline SiteDiv site_div(const Geo& g) { return {fast_div(g.L3h), fast_div(g.L2), fast_div(g.L1), fast_div(g.V3h)}; }

__device__ __forceinline__ int fdiv(FastDiv d, int n) {
  return (int)(((unsigned long long)(unsigned)n * d.m) >> d.s);
}

// the neighbour of site j of parity p in direction MU (DIR 0 forward, 1 backward), and the
// x0 of the site where MU = 0
template <int MU, int DIR>
__device__ __forceinline__ int nbr32(const Geo& g, const SiteDiv& q, int p, int j, int& x0) {
  const int r = fdiv(q.d3, j), x3h = j - r * g.L3h;
  x0 = 0;
  if constexpr (MU == 0) {
    x0 = fdiv(q.dv, j);
    if (DIR == 0) return x0 == g.L0 - 1 ? j - (g.L0 - 1) * g.V3h : j + g.V3h;
    return x0 == 0 ? j + (g.L0 - 1) * g.V3h : j - g.V3h;
  } else {
    const int r2 = fdiv(q.d2, r), x2 = r - r2 * g.L2;
    if constexpr (MU == 2) {
      if (DIR == 0) return x2 == g.L2 - 1 ? j - (g.L2 - 1) * g.L3h : j + g.L3h;
      return x2 == 0 ? j + (g.L2 - 1) * g.L3h : j - g.L3h;
    } else {
      const int r3 = fdiv(q.d1, r2), x1 = r2 - r3 * g.L1;
      const int st = g.L2 * g.L3h;
      if constexpr (MU == 1) {
        if (DIR == 0) return x1 == g.L1 - 1 ? j - (g.L1 - 1) * st : j + st;
        return x1 == 0 ? j + (g.L1 - 1) * st : j - st;
      } else {
        const int b = (p + r3 + x1 + x2) & 1;
        if (DIR == 0) {
          const int h = x3h + b;
          return j + b - (h == g.L3h ? g.L3h : 0);
        }
        const int h = x3h - 1 + b;
        return j - 1 + b + (h < 0 ? g.L3h : 0);
      }
    }
  }
}

// the launch's x0 ranges (nblk of Vb sites per parity, nchunk workgroups of 64 sites each)
// and the divisors of the site decomposition
struct SplitGeo {
  int nblk, len, Vb, nchunk;
  int nslice, npiece;   // marching order: 64-site chunks of a slice, and at most of an XCD's share
  SiteDiv site;
  FastDiv db;           // the block length
};

// does the launch leave out some of the x0 blocks?
template <class R> inline bool split_partial(const HopArgs<R>& A) {
  return A.slb && (A.block >= 0 || A.colour != 0);
}

// 64-site workgroups of one system of nlb x0 slices (0: the full lattice): the partials of
// its fused reductions
int split_chunks(const Geo& g, int nlb, bool march);

template <class R> void launch_split(const HopArgs<R>& A, bool march, hipStream_t st);

}  // namespace sap
