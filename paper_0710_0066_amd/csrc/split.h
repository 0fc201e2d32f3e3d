// The hop kernel that spreads the eight hops of a site over a workgroup (split.hip).
#pragma once
#include "internal.h"

namespace sap {

// division of 0 <= n < 2^31 by a divisor known at launch: (n * m) >> s
struct FastDiv {
  unsigned m;
  int s;
};

// the launch's x0 ranges (nblk of Vb sites per parity, nchunk workgroups of 64 sites each)
// and the divisors of the site decomposition (L3 / 2, L2, L1, V3h, and the block length)
struct SplitGeo {
  int nblk, len, Vb, nchunk;
  int nslice, npiece;   // marching order: 64-site chunks of a slice, and at most of an XCD's share
  FastDiv d3, d2, d1, dv, db;
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
