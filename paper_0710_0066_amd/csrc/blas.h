// Declarations of the BLAS-1 / reduction launchers (blas.hip) used by the solvers.
#pragma once
#include <algorithm>
#include "internal.h"

namespace sap {

// Systems of a batched solve: nblk x0 blocks of Vb sites per parity (nblk = 1, Vb = Vh
// for the full lattice), selection of the blocks (block_selected code: 0 all, 1 black,
// 2 white, 3 + b block b).
struct SysGrid {
  int nblk;
  long long Vb;
  int per;          // sites per workgroup of the BLAS kernels, a multiple of 64
  int nchunk;       // ceil(Vb / per)
  int colour;
  int nrhs;
  bool xcd;         // workgroups in the order of the split hop (tile_of)
  long long Vh;
  long long Vhp;     // storage sites per parity (locates the site norms of FP16 fields)
};

// Per-system scalars and flags. The kernels of an iteration form the scalars they need
// from the partial sums themselves (every workgroup of a system the same value); the first
// workgroup of a system records the new state. As the others may still read the old one,
// gam, active and cs hold two versions of nsys entries each, and a kernel that steps the
// state reads version v and writes version 1 - v.
// flags[0] = non-finite value seen (1 CG init, 2 CG alpha, 3 CG beta, 4 BiCGstab rho, 5
// BiCGstab alpha, 6 BiCGstab omega, 7 series), flags[1] = number of active systems, flags[2] = a
// geometric series diverged.
struct SysScal {
  double *gam, *ss, *alpha;
  double* cs;           // BiCGstab: complex (rho, alpha, omega, beta) per system
  int *active, *iters, *flags;
  const int* selected;
  const double* target2;
  int nsys;
  int rev = 0;          // walk the systems' sites backwards
};

// partial sums: n per system (of one value, or of three interleaved), system-major
struct Parts {
  const double* p;
  int n;
};

// Sites per workgroup: 64 while that gives up to about a thousand workgroups, then more, up to
// 1024, and above that as many as keep a system at a thousand chunks (its partials are summed
// again by every workgroup that needs the scalar). On 16^3x32 with one rhs a CG update takes 3 to
// 4 us with 64 sites per workgroup, 6.4 to 9 us with the 1024 that suit 12 rhs on 24^3x48 (64
// workgroups on 256 CUs). FP16 kernels take a site per work-item and keep at least 256.
// ranges: the hops of the solve give each XCD a range of the whole lattice (hop_in_ranges), so that
// the updates may follow them. CG solves with it / without (ms): 16^3x32 1 rhs FP32 3.81 / 3.89,
// FP64 5.69 / 5.75, FP16 blocks 2.93 / 3.04; 16x12^3 2 rhs FP32 2.31 / 2.38. Below 25000 sites times
// rhs the index divisions cost more, above 200000 nothing is gained (16^3x32 5 rhs, FP64 1% lost).
inline SysGrid make_sysgrid(long long Vh, int V3h, int lb, int L0, int colour, int nrhs, bool f16 = false,
                            bool ranges = false) {
  SysGrid G;
  G.nblk = lb ? L0 / lb : 1;
  G.Vb = lb ? (long long)lb * V3h : Vh;
  const long long tiles = (G.Vb + TILE - 1) / TILE * G.nblk * nrhs;
  G.per = TILE * (int)std::max(std::min(16LL, std::max(f16 ? 4LL : 1LL, tiles / 1024)), (G.Vb / TILE + 1023) / 1024);
  G.nchunk = (int)((G.Vb + G.per - 1) / G.per);
  G.colour = lb ? colour : 0;
  G.nrhs = nrhs;
  G.xcd = ranges && Vh * nrhs > 25000 && Vh * nrhs <= 200000;
  G.Vh = Vh;
  G.Vhp = (Vh + TILE - 1) / TILE * TILE;
  return G;
}

// ||a||^2 over npar parities: npar * nchunk partials per system
template <class R> void blas_norm2(const SysGrid& G, int nrhs, Field<R> a, int npar, double* part, hipStream_t s);
// alpha = gam / ||q||^2 from its partials; s -= alpha q with partial ||s||^2 (state read at v)
template <class R> void blas_cg_s(const SysGrid& G, int nrhs, Field<R> sf, Field<R> q, const SysScal& S, int v,
                                  Parts qq, double* part, hipStream_t s);
// beta = ||r||^2 / gam and the convergence test on ||s||^2 from their partials (state v to
// 1 - v); x += alpha p, then p = r + beta p
template <class R> void blas_cg_xp(const SysGrid& G, int nrhs, Field<R> x, Field<R> p, Field<R> r, const SysScal& S,
                                   int v, Parts ss, Parts rr, hipStream_t s);
// out = scale * in on the even sites at another precision, partial ||out||^2
template <class R> void blas_convert(const SysGrid& G, int nrhs, Field<R> out, Field<double> in, double scale,
                                     double* part, hipStream_t s);
// even sites of the selected systems: x += e (e at another precision), w = b - aI x
template <class R> void blas_add_resid(const SysGrid& G, int nrhs, Field<double> x, Field<R> e, Field<double> b,
                                       Field<double> w, double aI, hipStream_t s);

// ---- sums of partials, one wavefront per system in a fixed order
void fin_sum(int nsys, Parts a, double* out, hipStream_t s);
// out[3 * sys + k] = the three sums
void fin_sum3(int nsys, Parts a, double* out, hipStream_t s);
// target2 = max(inner2 ||b_hat||^2, abs2 bnorm2)
void fin_targets(int nsys, Parts bh, const double* bnorm2, double inner2, double abs2, double* target2, hipStream_t s);
// fewer partials: sums of 256 neighbouring ones (nv values each); returns the new count
int compress_parts(int nsys, int nv, Parts a, double* out, hipStream_t s);
// start of an inner CG (state version 0) from ||b_hat||^2 and ||r||^2
void fin_init(const SysScal& S, Parts b, Parts r, hipStream_t s);
// number of active systems of version v into flags[1]
void fin_count(const SysScal& S, int v, hipStream_t s);

// ---- BiCGstab on the even-odd system: complex per-system scalars in cs[8 * sys] =
// (rho, alpha, omega, beta) as (re, im) pairs; partials hold three values: re <a, b>,
// im <a, b>, ||c||^2.
template <class R> void blas_cdot3(const SysGrid& G, int nrhs, Field<R> a, Field<R> b, Field<R> c, double* part,
                                   hipStream_t s);
// p = r + beta (p - omega v); rho.p: first close the previous iteration from its partials
// <r0, r>, ||r||^2 (fin_bicg_rho; state v to 1 - v)
template <class R> void blas_bicg_p(const SysGrid& G, int nrhs, Field<R> p, Field<R> r, Field<R> v, const SysScal& S,
                                    int ver, Parts rho, hipStream_t s);
// alpha = rho / <r0, v> (state v to 1 - v); s = r - alpha v (into r), partial ||s||^2
template <class R> void blas_bicg_s(const SysGrid& G, int nrhs, Field<R> r, Field<R> v, const SysScal& S, int ver,
                                    Parts den, double* part, hipStream_t s);
// omega = <t, s> / ||t||^2 (state v to 1 - v); x += alpha p + omega s ; r = s - omega t (s is
// held in r) ; partials <r0, r>, ||r||^2
template <class R> void blas_bicg_xr(const SysGrid& G, int nrhs, Field<R> x, Field<R> p, Field<R> r,
                                     Field<R> t, Field<R> r0, const SysScal& S, int ver, Parts ts, Parts ss,
                                     double* part, hipStream_t s);
// start (init: writes version 0) or close an iteration (state v to 1 - v): rho_new = <r0, r>,
// convergence on ||r||^2, beta; counts the active systems
void fin_bicg_rho(const SysScal& S, int ver, Parts a, int init, hipStream_t s);

// y = c0 y + c1 u + c2 w (w.ptr may be null; y is not read when c0 = 0) with complex
// per-system coefficients
// coef[6 * sys] = (c0, c1, c2); if part: partials <q, y>, ||y||^2 (three per chunk)
template <class R> void blas_lin3(const SysGrid& G, int nrhs, Field<R> y, Field<R> u, Field<R> w, Field<R> q,
                                  const double* coef, double* part, hipStream_t s);

// ---- geometric series: x += t on active systems; tt.p: first test the term from the
// partials ||t||^2 (fin_geom; state v to 1 - v)
template <class R> void blas_geom_add(const SysGrid& G, int nrhs, Field<R> x, Field<R> t, const SysScal& S, int ver,
                                      Parts tt, hipStream_t s);
// start (init: writes version 0) or test a term (flags[2] = 1 when a series diverges);
// counts the active systems
void fin_geom(const SysScal& S, int ver, Parts tt, int init, hipStream_t s);

}  // namespace sap
