// Conversions between the canonical interchange layout (lexicographic sites,
// array-of-structures complex128) and the library's even-odd structure-of-arrays
// layout. One work-item per site (and rhs); not on the hot path.
#include "internal.h"
#include "link_copies.h"

namespace sap {

struct Lex {
  int x0, x1, x2, x3;
};

__device__ __forceinline__ Lex lex_coords(const Geo& g, long long i) {
  Lex c;
  c.x3 = (int)(i % g.L3); i /= g.L3;
  c.x2 = (int)(i % g.L2); i /= g.L2;
  c.x1 = (int)(i % g.L1);
  c.x0 = (int)(i / g.L1);
  return c;
}

template <class R>
__global__ void pack_spinor_kernel(Geo g, typename vec2<R>::type* out, const double2* in, int nrhs) {
  const long long V = 2 * g.Vh;
  const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= V * nrhs) return;
  const long long rhs = t / V, i = t - rhs * V;
  const Lex c = lex_coords(g, i);
  const int p = (c.x0 + c.x1 + c.x2 + c.x3) & 1;
  const long long j = i >> 1;
  typename vec2<R>::type* o = out + (rhs * 2 + p) * 12 * g.Vhp;
  const double2* src = in + (rhs * V + i) * 12;
  for (int k = 0; k < 12; ++k) {
    double2 v = src[k];
    typename vec2<R>::type w;
    w.x = (R)v.x; w.y = (R)v.y;
    o[sidx<R>(j, k)] = w;
  }
}

template <class R>
__global__ void unpack_spinor_kernel(Geo g, double2* out, const typename vec2<R>::type* in, int nrhs) {
  const long long V = 2 * g.Vh;
  const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= V * nrhs) return;
  const long long rhs = t / V, i = t - rhs * V;
  const Lex c = lex_coords(g, i);
  const int p = (c.x0 + c.x1 + c.x2 + c.x3) & 1;
  const long long j = i >> 1;
  const typename vec2<R>::type* src = in + (rhs * 2 + p) * 12 * g.Vhp;
  double2* o = out + (rhs * V + i) * 12;
  for (int k = 0; k < 12; ++k) {
    typename vec2<R>::type v = src[sidx<R>(j, k)];
    o[k] = make_double2((double)v.x, (double)v.y);
  }
}

// Canonical links (36 complex numbers per site, sites in lexicographic order) to and from the
// tiled layout through LDS: a workgroup owns 64 neighbouring pairs of sites (2j, 2j + 1), one of
// each parity, a tile of both parities and 72 KB of consecutive memory. The canonical side
// moves in whole lines, 16 bytes per lane, and a work-item then holds one link (wavefront w:
// parity w & 1, direction w >> 1). Loading also writes the reduced copies and the workgroup's
// largest deviation from SU(3) (an entry of U U^+ - 1, or |det U - 1|; a NaN entry gives NaN).
// Both are bound by memory. With a work-item per site, whose 36 numbers lie 576 bytes from its
// neighbour's, the conversion took 317 us on 24^3x48 and storing 414 us; the copies (168 us)
// and the check (108 us) read the links again.
constexpr int LINK_PAIRS = 64;

// site of this work-item's link within the workgroup's 128 lexicographic sites
__device__ __forceinline__ int pair_site(const Geo& g, long long j, int p, int lane) {
  return 2 * lane + decode(g, j, p).b;
}

__global__ __launch_bounds__(512) void load_gauge_kernel(Geo g, double2* U64, LinkCopies lc, const double2* in,
                                                        double* part) {
  extern __shared__ double2 sl[];
  __shared__ double sh[8];
  const long long base = (long long)blockIdx.x * (2 * LINK_PAIRS) * 36, n = 2 * g.Vh * 36;
#pragma unroll
  for (int k = 0; k < 9; ++k) {
    const int i = threadIdx.x + 512 * k;
    if (base + i < n) sl[i] = in[base + i];
  }
  __syncthreads();
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, p = w & 1, mu = w >> 1;
  const long long j = (long long)blockIdx.x * LINK_PAIRS + lane;
  double dev = 0.0;
  if (j < g.Vh) {
    const double2* u = sl + pair_site(g, j, p, lane) * 36 + 9 * mu;
    double2 e[9];
    cx<double> m[9];
#pragma unroll
    for (int k = 0; k < 9; ++k) {
      e[k] = u[k];
      m[k] = {e[k].x, e[k].y};
      U64[p * 36 * g.Vhp + tiled(j, 9 * mu + k, 36)] = e[k];
    }
    write_link_copies(lc, g.Vhp, p, j, mu, e);
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
      for (int b = 0; b < 3; ++b) {
        cx<double> t = cmulj(m[3 * a], m[3 * b]) + cmulj(m[3 * a + 1], m[3 * b + 1]) + cmulj(m[3 * a + 2], m[3 * b + 2]);
        const double re = t.r - (a == b ? 1.0 : 0.0);
        dev = nanmax(dev, sqrt(re * re + t.i * t.i));
      }
    // det = row 0 . (row 1 x row 2)
    const cx<double> c0 = cmul(m[4], m[8]) - cmul(m[5], m[7]);
    const cx<double> c1 = cmul(m[5], m[6]) - cmul(m[3], m[8]);
    const cx<double> c2 = cmul(m[3], m[7]) - cmul(m[4], m[6]);
    const cx<double> det = cmul(m[0], c0) + cmul(m[1], c1) + cmul(m[2], c2);
    dev = nanmax(dev, sqrt((det.r - 1.0) * (det.r - 1.0) + det.i * det.i));
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) dev = nanmax(dev, __shfl_down(dev, off, 64));
  if (lane == 0) sh[w] = dev;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int k = 1; k < 8; ++k) dev = nanmax(dev, sh[k]);
    part[blockIdx.x] = dev;
  }
}

__global__ __launch_bounds__(512) void unpack_gauge_kernel(Geo g, double2* out, const double2* U64) {
  extern __shared__ double2 sl[];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, p = w & 1, mu = w >> 1;
  const long long j = (long long)blockIdx.x * LINK_PAIRS + lane;
  if (j < g.Vh) {
    double2* u = sl + pair_site(g, j, p, lane) * 36 + 9 * mu;
#pragma unroll
    for (int k = 0; k < 9; ++k) u[k] = U64[p * 36 * g.Vhp + tiled(j, 9 * mu + k, 36)];
  }
  __syncthreads();
  const long long base = (long long)blockIdx.x * (2 * LINK_PAIRS) * 36, n = 2 * g.Vh * 36;
#pragma unroll
  for (int k = 0; k < 9; ++k) {
    const int i = threadIdx.x + 512 * k;
    if (base + i < n) out[base + i] = sl[i];
  }
}

// FP32 / FP16 link copies keep the first two rows of each link (6 of 9 entries, component
// c = 6 mu + e). The FP32 copy stores the entries of a tile row in pairs
// (2k, 2k + 1) of one link, one 16-byte word per lane:
//   p*24*Vhp + (j / 64)*24*64 + (c - c % 2)*64 + 2*(j % 64) + c % 2,
// so that a link is three 16-byte loads per work-item. The FP16 copy stores the six
// entries of a link of a tile row as a quad (e = 0..3, one 16-byte word per lane) and a
// pair (e = 4, 5, 8 bytes per lane):
//   p*24*Vhp + (j / 64)*24*64 + 6 mu*64 + (e < 4 ? 4*(j % 64) + e : 256 + 2*(j % 64) + e - 4),
// two loads per link. The LDS-staged FP16 hop, with one rhs per work-item, reads a
// three-row copy instead, so that it does not rebuild the third row for every term: after
// the two-row copy (at U16 + 48*Vhp) it holds all nine entries of a link of a tile row as
// two quads (e = 0..3, 4..7) and a single entry,
//   p*36*Vhp + (j / 64)*36*64 + 9 mu*64 + (e < 4 ? 4*(j % 64) + e : e < 8 ? 256 + 4*(j % 64) + e - 4 : 512 + j % 64),
// each entry rounded from the FP64 link (the third row is not rebuilt from rounded rows).
// internal.h (write_link_copies) writes all copies of one link; this kernel runs it with
// one work-item per link (site j fastest).
__global__ void gauge_to_f32_kernel(long long Vhp, LinkCopies lc, const double2* U64) {
  const long long k = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= 8 * Vhp) return;
  const long long j = k % Vhp, r = k / Vhp;
  const int mu = (int)(r % 4), p = (int)(r / 4);
  double2 e[9];
#pragma unroll
  for (int c = 0; c < 9; ++c) e[c] = U64[p * 36 * Vhp + tiled(j, 9 * mu + c, 36)];
  write_link_copies(lc, Vhp, p, j, mu, e);
}

// FP16 spinor fields: components divided by the site norm (the largest component
// magnitude), in quads of components (sidx), norm in FP32 (rhs blocks of 26*Vhp
// four-byte entries)
__global__ void pack_spinor16_kernel(Geo g, __half2* out, const double2* in, int nrhs) {
  const long long V = 2 * g.Vh;
  const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= V * nrhs) return;
  const long long rhs = t / V, i = t - rhs * V;
  const Lex c = lex_coords(g, i);
  const int p = (c.x0 + c.x1 + c.x2 + c.x3) & 1;
  const long long j = i >> 1;
  __half2* blk = out + rhs * 26 * g.Vhp;
  const double2* src = in + (rhs * V + i) * 12;
  float m = 0.0f;
  for (int k = 0; k < 12; ++k) m = fmaxf(m, fmaxf(fabsf((float)src[k].x), fabsf((float)src[k].y)));
  const float inv = m > 0.0f ? 1.0f / m : 0.0f;
  for (int k = 0; k < 12; ++k)
    blk[p * 12 * g.Vhp + sidx<h16>(j, k)] = __floats2half2_rn((float)src[k].x * inv, (float)src[k].y * inv);
  ((float*)(blk + 24 * g.Vhp))[p * g.Vhp + j] = m;
}

__global__ void unpack_spinor16_kernel(Geo g, double2* out, const __half2* in, int nrhs) {
  const long long V = 2 * g.Vh;
  const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= V * nrhs) return;
  const long long rhs = t / V, i = t - rhs * V;
  const Lex c = lex_coords(g, i);
  const int p = (c.x0 + c.x1 + c.x2 + c.x3) & 1;
  const long long j = i >> 1;
  const __half2* blk = in + rhs * 26 * g.Vhp;
  const float m = ((const float*)(blk + 24 * g.Vhp))[p * g.Vhp + j];
  double2* o = out + (rhs * V + i) * 12;
  for (int k = 0; k < 12; ++k) {
    const float2 v = __half22float2(blk[p * 12 * g.Vhp + sidx<h16>(j, k)]);
    o[k] = make_double2((double)(v.x * m), (double)(v.y * m));
  }
}

__global__ void pack_momenta_kernel(Geo g, double* out, const double* in, int to_sap) {
  const long long V = 2 * g.Vh;
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= V) return;
  const Lex c = lex_coords(g, i);
  const int p = (c.x0 + c.x1 + c.x2 + c.x3) & 1;
  const long long j = i >> 1;
  for (int mu = 0; mu < 4; ++mu)
    for (int a = 0; a < 8; ++a) {
      long long ks = p * 32 * g.Vhp + tiled(j, 8 * mu + a, 32);
      long long kc = (i * 4 + mu) * 8 + a;
      if (to_sap) out[ks] = in[kc];
      else out[kc] = in[ks];
    }
}

static inline unsigned nblk(long long n, int b) { return (unsigned)((n + b - 1) / b); }

template <class R>
void launch_pack_spinor(const Geo& g, typename vec2<R>::type* out, const double2* in, int nrhs,
                        hipStream_t s) {
  long long n = 2 * g.Vh * nrhs;
  hipLaunchKernelGGL(pack_spinor_kernel<R>, dim3(nblk(n, 256)), dim3(256), 0, s, g, out, in, nrhs);
}
template <class R>
void launch_unpack_spinor(const Geo& g, double2* out, const typename vec2<R>::type* in, int nrhs,
                          hipStream_t s) {
  long long n = 2 * g.Vh * nrhs;
  hipLaunchKernelGGL(unpack_spinor_kernel<R>, dim3(nblk(n, 256)), dim3(256), 0, s, g, out, in, nrhs);
}
template void launch_pack_spinor<double>(const Geo&, double2*, const double2*, int, hipStream_t);
template void launch_pack_spinor<float>(const Geo&, float2*, const double2*, int, hipStream_t);
template void launch_unpack_spinor<double>(const Geo&, double2*, const double2*, int, hipStream_t);
template void launch_unpack_spinor<float>(const Geo&, double2*, const float2*, int, hipStream_t);

constexpr size_t LINK_LDS = (size_t)2 * LINK_PAIRS * 36 * sizeof(double2);
int load_gauge_parts(const Geo& g) { return (int)nblk(g.Vh, LINK_PAIRS); }
void launch_load_gauge(const Geo& g, double2* U64, float2* U32, __half2* U16, const double2* in, double* part,
                       hipStream_t s) {
  hipLaunchKernelGGL(load_gauge_kernel, dim3(load_gauge_parts(g)), dim3(512), LINK_LDS, s, g, U64,
                     LinkCopies{U32, U16}, in, part);
}
void launch_unpack_gauge(const Geo& g, double2* out, const double2* U64, hipStream_t s) {
  hipLaunchKernelGGL(unpack_gauge_kernel, dim3(load_gauge_parts(g)), dim3(512), LINK_LDS, s, g, out, U64);
}
void launch_gauge_to_f32(const Geo& g, float2* U32, __half2* U16, const double2* U64, hipStream_t s) {
  const long long n = 8LL * g.Vhp;   // links: 2 parities x Vhp sites x 4 directions
  hipLaunchKernelGGL(gauge_to_f32_kernel, dim3(nblk(n, 256)), dim3(256), 0, s, g.Vhp, LinkCopies{U32, U16}, U64);
}
void launch_pack_spinor16(const Geo& g, __half2* out, const double2* in, int nrhs, hipStream_t s) {
  long long n = 2 * g.Vh * nrhs;
  hipLaunchKernelGGL(pack_spinor16_kernel, dim3(nblk(n, 256)), dim3(256), 0, s, g, out, in, nrhs);
}
void launch_unpack_spinor16(const Geo& g, double2* out, const __half2* in, int nrhs, hipStream_t s) {
  long long n = 2 * g.Vh * nrhs;
  hipLaunchKernelGGL(unpack_spinor16_kernel, dim3(nblk(n, 256)), dim3(256), 0, s, g, out, in, nrhs);
}
void launch_pack_momenta(const Geo& g, double* out, const double* in, hipStream_t s) {
  hipLaunchKernelGGL(pack_momenta_kernel, dim3(nblk(2 * g.Vh, 128)), dim3(128), 0, s, g, out, in, 1);
}
void launch_unpack_momenta(const Geo& g, double* out, const double* in, hipStream_t s) {
  hipLaunchKernelGGL(pack_momenta_kernel, dim3(nblk(2 * g.Vh, 128)), dim3(128), 0, s, g, out, in, 0);
}

}  // namespace sap
