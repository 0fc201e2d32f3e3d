// Wilson hop with the eight hops of a site spread over the eight wavefronts of a workgroup
// (Sec. 1, eq. 2; the operator of dslash.hip and half.hip, every storage precision).
//
// With one work-item per site a small lattice leaves the chip short of wavefronts (16^3 x 32
// has 1024 wavefronts of sites per parity and right-hand side, one per SIMD), and a launch
// takes the latency of eight dependent rounds of loads. Here a workgroup owns 64
// consecutive sites of one parity of one x0 range for one right-hand side, wavefront w
// computes hop w (mu = w / 2, forward or backward), so that mu and the direction are uniform
// over the wavefront and all loads of a site are in flight at once, and writes its half
// spinor (two colour vectors) to LDS; after one barrier wavefronts 0..5 sum the eight hops
// of a pair of components each (spin-colour components 2k, 2k + 1), form a x + b D in and
// store the pair. 50 / 92 VGPRs (FP32 / FP64) instead of 128 and more leave 8 / 4 wavefronts
// per SIMD (workgroups of two per SIMD become resident whole). FP16 fields run the linear order
// only: where their launches are large enough to march, one work-item per site is faster (half.hip).
// What bounds it: memory latency up to about 10^4 sites, then L2 / MALL bandwidth (the links
// and the eight-fold gather of the input). Measured per launch against one work-item per
// site (us): half hop on 16x8^3, FP64 4.5 / 12.7, FP32 3.9 / 7.5; on 16^3x32, FP64 15.2 / 20.4, FP32
// 7.4 / 9.7, FP32 with 12 rhs 48 / 92; apply_M FP64 on 16^3x32 23.3 / 40 (5.4 TB/s of its
// algorithmic bytes), on 24^3x48 133 / 226 in the marching order.
#include "site_io.h"
#include "split.h"

namespace sap {

namespace {

// half spinor of hop (MU, DIR) of site j, zero where the hop is absent
template <class R, int MU, int DIR>
__device__ __forceinline__ void split_hop(const HopArgs<R>& A, const SplitGeo& q, int rhs, int p, int j, bool on,
                                          cx<arith_t<R>> w[6]) {
  typedef arith_t<R> T;
  const Geo& g = A.g;
  const long long Vhp = g.Vhp;
  int x0;
  const int jn = nbr32<MU, DIR>(g, q.site, p, j, x0);
  bool flip = false;
  if constexpr (MU == 0) {
    flip = DIR == 0 ? x0 == g.L0 - 1 : x0 == 0;
    if (A.lb) {
      const int r = x0 - fdiv(q.db, x0) * A.lb;
      on = on && (DIR == 0 ? r != A.lb - 1 : r != 0);
    }
  }
#pragma unroll
  for (int k = 0; k < 6; ++k) w[k] = {T(0), T(0)};
  if (!on) return;
  const bool g5i = A.g5_in != 0;
  const int lp = DIR == 0 ? p : 1 - p, lj = DIR == 0 ? j : jn;    // parity and site of the link
  if constexpr (is_h16<R>) {
    const SiteR<h16> in = site_r(A.in, rhs, 1 - p, jn, Vhp);
    unsigned e[9], sw[12];
    load_link16_words(A.U + lp * 24 * Vhp + (long long)(lj >> 6) * (24 * TILE) + 6 * MU * TILE, lj & 63, e);
    third_row16(e);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const u4v v = *(const u4v*)(in.b + 4 * k * TILE);
      sw[4 * k] = v.x; sw[4 * k + 1] = v.y; sw[4 * k + 2] = v.z; sw[4 * k + 3] = v.w;
    }
    cx<float> uh[2][3];
    if (g5i) hop16_term<true>(MU, DIR == 1, e, sw, uh);
    else hop16_term<false>(MU, DIR == 1, e, sw, uh);
    const float m = flip ? -in.m : in.m;
#pragma unroll
    for (int k = 0; k < 6; ++k) w[k] = m * uh[k / 3][k % 3];
  } else {
    cx<T> v[12], s[4][3], h[2][3], m[9];
    ld_site<R>(A.in.ptr + rhs * A.in.rs + (1 - p) * A.in.ps, jn, v);
    if constexpr (is_f32<R>) {
      const f4v* u = (const f4v*)(A.U + lp * 24 * Vhp) + tiled(lj, 3 * MU, 12);
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        const f4v t = u[k * TILE];
        m[2 * k] = {t.x, t.y};
        m[2 * k + 1] = {t.z, t.w};
      }
    } else {
      const double2* u = A.U + lp * 36 * Vhp + tiled(lj, 9 * MU, 36);
#pragma unroll
      for (int k = 0; k < 6; ++k) m[k] = ld<R>(u + k * TILE);
    }
    third_row<T>(m);
#pragma unroll
    for (int k = 0; k < 12; ++k) s[k / 3][k % 3] = (g5i && k >= 6) ? -v[k] : v[k];
    project<T>(MU, DIR == 1, s, h);
    cx<T> uh[2][3];
    if (DIR == 0) {
      su3_mul<T>(m, h[0], uh[0]);
      su3_mul<T>(m, h[1], uh[1]);
    } else {
      su3_dag_mul<T>(m, h[0], uh[0]);
      su3_dag_mul<T>(m, h[1], uh[1]);
    }
#pragma unroll
    for (int k = 0; k < 6; ++k) w[k] = flip ? -uh[k / 3][k % 3] : uh[k / 3][k % 3];
  }
}

// component C = 3 spin + colour of the sum over the hops from their half spinors in LDS
// (device_common.h, accum_recon): upper spins add the half spinors, lower spins add them
// with the phases of the projection
template <class T, int C>
__device__ __forceinline__ cx<T> split_sum(const typename vec2<T>::type* g, int lane) {
  constexpr int sp = C / 3, c = C % 3, h = sp & 1;
  auto at = [&](int d, int hh) { return ld<T>(g + (d * 6 + 3 * hh + c) * TILE + lane); };
  cx<T> a = {T(0), T(0)};
#pragma unroll
  for (int d = 0; d < 8; ++d) {
    const int mu = d >> 1;
    const bool plus = d & 1;
    if (sp < 2) {
      a = a + at(d, h);
    } else if (mu == 0) {
      a = plus ? a - at(d, h) : a + at(d, h);
    } else if (mu == 1) {
      a = plus ? a + times_i(at(d, 1 - h)) : a - times_i(at(d, 1 - h));
    } else if (mu == 2) {
      a = plus == (h == 0) ? a + at(d, 1 - h) : a - at(d, 1 - h);
    } else {
      a = plus == (h == 0) ? a + times_i(at(d, h)) : a - times_i(at(d, h));
    }
  }
  return a;
}

template <class R, bool FULL, int RED, bool MARCH>
__global__ __launch_bounds__(512) void hop_split_kernel(HopArgs<R> A, SplitGeo q) {
  typedef arith_t<R> T;
  typedef typename vec2<T>::type T2;
  __shared__ T2 half[8 * 6 * TILE];
  __shared__ float mx[is_h16<R> ? 6 * TILE : 1];
  __shared__ double rsum[RED ? 6 * 3 : 1];
  const Geo& g = A.g;
  const long long Vhp = g.Vhp;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // workgroup: right-hand side fastest, then parity, 64-site chunk, x0 range (MARCH: slice)
  int rhs, p = A.parity_out, blk, ck, off, j;
  bool valid;
  if constexpr (MARCH) {
    // XCD k (workgroup id % 8) owns the chunks [nslice k / 8, nslice (k + 1) / 8) of every
    // slice and walks the slices in order
    const int xcd = blockIdx.x & 7;
    int w = blockIdx.x >> 3;
    rhs = w % A.nrhs;
    w /= A.nrhs;
    if (FULL) {
      p = w & 1;
      w >>= 1;
    }
    const int lo = q.nslice * xcd / 8, hi = q.nslice * (xcd + 1) / 8, x = w / q.npiece;
    const int cs = lo + w - x * q.npiece;
    if (cs >= hi || x >= g.L0) return;             // whole workgroup
    blk = x / q.len;
    ck = (x - blk * q.len) * q.nslice + cs;
    off = cs * TILE + lane;
    valid = off < g.V3h;
    j = x * g.V3h + (valid ? off : g.V3h - 1);
  } else {
    int w = xcd_block(blockIdx.x, gridDim.x, A.rev != 0);
    rhs = w % A.nrhs;
    w /= A.nrhs;
    if (FULL) {
      p = w & 1;
      w >>= 1;
    }
    blk = w / q.nchunk;
    ck = w - blk * q.nchunk;
    if (blk >= q.nblk) return;                     // whole workgroup: padding of the grid
    off = ck * TILE + lane;
    valid = off < q.Vb;
    j = blk * q.Vb + (valid ? off : q.Vb - 1);
  }
  if (A.active && !A.active[rhs * q.nblk + blk]) return;         // whole workgroup
  bool sel = true;
  if (A.slb) sel = A.block >= 0 ? blk == A.block : block_sel(blk, 1, -1, A.colour);
  if (A.keep && !sel) return;                                    // whole workgroup

  if (sel) {
    cx<T> v[6];
#define SAP_SPLIT(D) case D: split_hop<R, D / 2, D & 1>(A, q, rhs, p, j, valid, v); break;
    switch (wave) {
      SAP_SPLIT(0) SAP_SPLIT(1) SAP_SPLIT(2) SAP_SPLIT(3) SAP_SPLIT(4) SAP_SPLIT(5) SAP_SPLIT(6)
      default: split_hop<R, 3, 1>(A, q, rhs, p, j, valid, v); break;
    }
#undef SAP_SPLIT
#pragma unroll
    for (int k = 0; k < 6; ++k) st<T>(half + (wave * 6 + k) * TILE + lane, v[k]);
  }
  __syncthreads();

  cx<T> v[2] = {{T(0), T(0)}, {T(0), T(0)}}, xv[2] = {{T(0), T(0)}, {T(0), T(0)}};
  const int k2 = 2 * wave;                         // first component of this wavefront's pair
  if (wave < 6 && sel) {
    if (A.x.ptr) {
      const typename vec2<R>::type* xb = A.x.ptr + rhs * A.x.rs + p * A.x.ps + sidx<R>(j, k2);
      if constexpr (is_h16<R>) {
        const float m = norm_ptr16(A.x, rhs, p, Vhp)[j];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          const float2 f = __half22float2(xb[i]);
          xv[i] = {f.x * m, f.y * m};
        }
      } else if constexpr (is_f32<R>) {
        const f4v f = *(const f4v*)xb;
        xv[0] = {f.x, f.y};
        xv[1] = {f.z, f.w};
      } else {
        xv[0] = ld<R>(xb);
        xv[1] = ld<R>(xb + TILE);
      }
    }
#define SAP_PAIR(K) case K: v[0] = split_sum<T, 2 * K>(half, lane); v[1] = split_sum<T, 2 * K + 1>(half, lane); break;
    switch (wave) {
      SAP_PAIR(0) SAP_PAIR(1) SAP_PAIR(2) SAP_PAIR(3) SAP_PAIR(4)
      default: v[0] = split_sum<T, 10>(half, lane); v[1] = split_sum<T, 11>(half, lane); break;
    }
#undef SAP_PAIR
    const T b = (A.g5_out && wave >= 3) ? -A.b : A.b;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      v[i] = b * v[i];
      if (A.x.ptr) v[i] = v[i] + A.a * xv[i];
    }
  }
  typename vec2<R>::type* ob = A.out.ptr + rhs * A.out.rs + p * A.out.ps + sidx<R>(j, k2);
  if constexpr (is_h16<R>) {
    if (wave < 6)
      mx[wave * TILE + lane] = fmaxf(fmaxf(fabsf(v[0].r), fabsf(v[0].i)), fmaxf(fabsf(v[1].r), fabsf(v[1].i)));
    __syncthreads();
    if (wave < 6 && valid) {
      float m = 0.0f;
#pragma unroll
      for (int k = 0; k < 6; ++k) m = fmaxf(m, mx[k * TILE + lane]);
      const float inv = m > 0.0f ? 1.0f / m : 0.0f;
      typedef unsigned u2w __attribute__((ext_vector_type(2)));
      const u2w o = {u_of(__floats2half2_rn(v[0].r * inv, v[0].i * inv)),
                     u_of(__floats2half2_rn(v[1].r * inv, v[1].i * inv))};
      *(u2w*)ob = o;
      if (wave == 0) norm_ptr16(A.out, rhs, p, Vhp)[j] = m;
    }
  } else if constexpr (is_f32<R>) {
    if (wave < 6 && valid) {
      const f4v o = {v[0].r, v[0].i, v[1].r, v[1].i};
      if (MARCH) __builtin_nontemporal_store(o, (f4v*)ob);
      else *(f4v*)ob = o;
    }
  } else {
    if (wave < 6 && valid) {
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const d2v o = {v[i].r, v[i].i};
        if (MARCH) __builtin_nontemporal_store(o, (d2v*)(ob + i * TILE));
        else *(d2v*)(ob + i * TILE) = o;
      }
    }
  }
  if constexpr (RED > 0) {
    // the sums over the workgroup of the values before any rounding to FP16 (invalid lanes
    // hold another site's values and add nothing)
    double s[3] = {0.0, 0.0, 0.0};
    if (wave < 6 && valid) {
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const double vr = v[i].r, vi = v[i].i;
        if constexpr (RED == 1) {
          s[0] += vr * vr + vi * vi;
        } else {
          const double xr = xv[i].r, xi = xv[i].i;
          s[0] += vr * xr + vi * xi;
          s[1] += vr * xi - vi * xr;
          s[2] += vr * vr + vi * vi;
        }
      }
    }
    constexpr int NV = RED == 1 ? 1 : 3;
    if (wave < 6)
#pragma unroll
      for (int i = 0; i < NV; ++i) {
        double t = s[i];
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) t += __shfl_down(t, o, 64);
        if (lane == 0) rsum[i * 6 + wave] = t;
      }
    __syncthreads();
    if (threadIdx.x < NV) {
      double t = 0.0;
#pragma unroll
      for (int k = 0; k < 6; ++k) t += rsum[threadIdx.x * 6 + k];
      A.npart[(((long long)rhs * q.nblk + blk) * q.nchunk + ck) * NV + threadIdx.x] = t;
    }
  }
}

}  // namespace

int split_chunks(const Geo& g, int nlb, bool march) {
  const long long Vb = (long long)(nlb ? nlb : g.L0) * g.V3h;
  if (march) return (nlb ? nlb : g.L0) * ((g.V3h + TILE - 1) / TILE);
  return (int)((Vb + TILE - 1) / TILE);
}

template <class R> void launch_split(const HopArgs<R>& A, bool march, hipStream_t st) {
  const Geo& g = A.g;
  const bool full = A.parity_out < 0;
  SplitGeo q;
  q.len = A.npart ? A.nlb : A.slb ? A.slb : g.L0;
  q.nblk = g.L0 / q.len;
  q.Vb = q.len * g.V3h;
  q.nchunk = split_chunks(g, q.len, march);
  q.nslice = (g.V3h + TILE - 1) / TILE;
  q.npiece = (q.nslice + 7) / 8;
  q.site = site_div(g);
  q.db = fast_div(A.lb ? A.lb : 1);
  const long long per = (long long)A.nrhs * (full ? 2 : 1);
  // linear order: a multiple of 8 workgroups gives each XCD a range of the lattice; where some
  // x0 blocks are left out, one more than that deals the workgroups over the XCDs one by one
  const long long n8 = (per * q.nblk * q.nchunk + 7) / 8 * 8;
  const long long n = march ? 8 * per * g.L0 * q.npiece : split_partial(A) ? n8 + 1 : n8;
  const dim3 grid((unsigned)n), blk(512);
#define SAP_SPLIT(FULL, RED)                                                                             \
  do {                                                                                                   \
    if constexpr (!is_h16<R>)                                                                            \
      if (march) {                                                                                       \
        hipLaunchKernelGGL((hop_split_kernel<R, FULL, RED, true>), grid, blk, 0, st, A, q);              \
        break;                                                                                           \
      }                                                                                                  \
    hipLaunchKernelGGL((hop_split_kernel<R, FULL, RED, false>), grid, blk, 0, st, A, q);                 \
  } while (0)
  if (full) SAP_SPLIT(true, 0);
  else if (A.npart && A.red == 1) SAP_SPLIT(false, 1);
  else if (A.npart && A.red == 3) SAP_SPLIT(false, 3);
  else SAP_SPLIT(false, 0);
#undef SAP_SPLIT
}

template void launch_split<double>(const HopArgs<double>&, bool, hipStream_t);
template void launch_split<float>(const HopArgs<float>&, bool, hipStream_t);
template void launch_split<h16>(const HopArgs<h16>&, bool, hipStream_t);

}  // namespace sap
