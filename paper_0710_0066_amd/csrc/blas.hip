// BLAS-1 kernels and per-system reductions for the batched Krylov solvers.
//
// A "system" is one (rhs, x0-block) pair: block b of length lb holds the sites
// j in [b*Vb, (b+1)*Vb) of each parity, Vb = lb * V3h (lb = L0 for the full lattice).
// Every kernel here runs on the grid (chunk, block, rhs) with G.per sites per workgroup,
// so a workgroup never straddles two systems. FP64 and FP32 kernels are six wavefronts,
// each streaming one pair of components of 64 consecutive sites at a time (16-byte words);
// FP16 kernels, which renormalise whole sites, take a site per work-item. Sums accumulate in
// FP64: per-thread partials -> wavefront shuffle tree -> LDS across the wavefronts -> one
// partial per workgroup.
//
// The scalars of an iteration (alpha, beta, omega, the convergence test) are formed by the
// kernel that first needs them: every workgroup of a system adds the system's partials in
// the same fixed order, and the first workgroup records the new state. This takes the
// single-workgroup finalize kernels out of the iteration, in which one work-item added
// up to hundreds of partials in sequence (4 to 11 us each on 16^3x32, of a 93 us CG iteration,
// and a launch gap). Everything is bitwise reproducible run to run.
#include "blas.h"
#include "site_io.h"

namespace sap {

namespace {

template <class R> constexpr int BT = is_h16<R> ? 256 : 384;   // work-items per workgroup

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
  return v;
}

// Sums of N values over the NT threads of a workgroup, valid in every thread. sh: N * NT / 64
// doubles not in use by other threads.
template <int NT, int N> __device__ __forceinline__ void block_sums(double v[N], double* sh) {
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
#pragma unroll
  for (int k = 0; k < N; ++k) {
    const double t = wave_sum(v[k]);
    if (lane == 0) sh[k * (NT / 64) + wid] = t;
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < N; ++k) {
    double t = 0.0;
#pragma unroll
    for (int w = 0; w < NT / 64; ++w) t += sh[k * (NT / 64) + w];
    v[k] = t;
  }
}

// this thread's share of the N interleaved sums of a system's partials
template <int NT, int N> __device__ __forceinline__ void thread_parts(Parts a, long long sys, double v[N]) {
#pragma unroll
  for (int k = 0; k < N; ++k) v[k] = 0.0;
  const double* q = a.p + sys * a.n * N;
  for (int i = threadIdx.x; i < a.n; i += NT)
#pragma unroll
    for (int k = 0; k < N; ++k) v[k] += q[i * N + k];
}

struct Tile {
  bool selected;
  int rhs, blk, p, chunk;
  long long j0, j1;   // site range of this workgroup within its parity
  long long sys;
  long long part;     // index of this workgroup's partial
};

// G.xcd: a one-dimensional grid, rhs fastest, then parity, chunk and block, each XCD a
// contiguous range walked forwards or (rev) backwards, the order of the split hop, whose
// outputs are then read by the XCD that wrote them. Else blockIdx = (chunk, block, rhs * npar +
// parity): on larger fields the first order streams no faster (24^3x48 with 12 rhs: 10% slower),
// on smaller ones the divisions cost more than they give, on some of the blocks it leaves XCDs
// without work (black blocks of 24x16^3, 2 rhs, FP64 CG: 3.95 ms, 3.57 without).
__device__ __forceinline__ Tile tile_of(const SysGrid& G, int npar = 1, bool rev = false) {
  Tile t;
  if (G.xcd) {
    int w = xcd_block(blockIdx.x, gridDim.x, rev);
    t.rhs = w % G.nrhs;
    w /= G.nrhs;
    t.p = npar == 1 ? 0 : w % npar;
    if (npar != 1) w /= npar;
    t.blk = w / G.nchunk;
    t.chunk = w - t.blk * G.nchunk;
  } else {
    t.chunk = blockIdx.x;
    t.blk = blockIdx.y;
    t.rhs = npar == 1 ? blockIdx.z : blockIdx.z / npar;
    t.p = npar == 1 ? 0 : blockIdx.z - t.rhs * npar;
  }
  t.sys = (long long)t.rhs * G.nblk + t.blk;
  t.selected = block_selected(G.colour, t.blk);
  t.j0 = (long long)t.blk * G.Vb + (long long)t.chunk * G.per;
  t.j1 = (long long)t.blk * G.Vb + G.Vb;
  if (t.j0 + G.per < t.j1) t.j1 = t.j0 + G.per;
  t.part = (t.sys * npar + t.p) * G.nchunk + t.chunk;
  return t;
}

// components 2w, 2w + 1 of site j (FP64, FP32)
template <class R>
__device__ __forceinline__ void ld_pair(const Field<R>& f, int rhs, int p, long long j, int w, cx<R> v[2]) {
  const typename vec2<R>::type* b = f.ptr + rhs * f.rs + p * f.ps + sidx<R>(j, 2 * w);
  if constexpr (is_f32<R>) {
    const f4v q = *(const f4v*)b;
    v[0] = {q.x, q.y};
    v[1] = {q.z, q.w};
  } else {
    v[0] = ld<R>(b);
    v[1] = ld<R>(b + TILE);
  }
}
template <class R>
__device__ __forceinline__ void st_pair(const Field<R>& f, int rhs, int p, long long j, int w, const cx<R> v[2]) {
  typename vec2<R>::type* b = f.ptr + rhs * f.rs + p * f.ps + sidx<R>(j, 2 * w);
  if constexpr (is_f32<R>) {
    *(f4v*)b = f4v{v[0].r, v[0].i, v[1].r, v[1].i};
  } else {
    st<R>(b, v[0]);
    st<R>(b + TILE, v[1]);
  }
}

// Streams the sites of a tile: fold() forms the scalars (it may synchronise; false: nothing
// to do), op(in, out) maps the NIN components of the input fields to the NOUT of the output
// fields. The first loads of a work-item are issued before fold, whose partial sums they
// overlap with.
template <class R, int NIN, int NOUT, class Fold, class Op>
__device__ __forceinline__ void stream(const Tile& t, long long Vhp, const Field<R> (&in)[NIN],
                                       const Field<R> (&out)[NOUT], Fold fold, Op op) {
  typedef arith_t<R> A;
  if constexpr (is_h16<R>) {
    if (!fold()) return;
    for (long long j = t.j0 + threadIdx.x; j < t.j1; j += BT<R>) {
      SiteR<R> r[NIN];
      SiteW<R> w[NOUT];
#pragma unroll
      for (int k = 0; k < NIN; ++k) r[k] = site_r(in[k], t.rhs, t.p, j, Vhp);
#pragma unroll
      for (int k = 0; k < NOUT; ++k) w[k] = site_w(out[k], t.rhs, t.p, j, Vhp);
#pragma unroll
      for (int c = 0; c < 12; ++c) {
        cx<A> v[NIN], o[NOUT];
#pragma unroll
        for (int k = 0; k < NIN; ++k) v[k] = get(r[k], c);
        op(v, o);
#pragma unroll
        for (int k = 0; k < NOUT; ++k) put(w[k], c, o[k]);
      }
#pragma unroll
      for (int k = 0; k < NOUT; ++k) close(w[k]);
    }
  } else {
    const int wv = threadIdx.x >> 6;
    long long j = t.j0 + (threadIdx.x & 63);
    cx<A> v[NIN][2];
    if (j < t.j1)
#pragma unroll
      for (int k = 0; k < NIN; ++k) ld_pair<R>(in[k], t.rhs, t.p, j, wv, v[k]);
    if (!fold()) return;
    while (j < t.j1) {
      cx<A> o[NOUT][2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        cx<A> vi[NIN], oi[NOUT];
#pragma unroll
        for (int k = 0; k < NIN; ++k) vi[k] = v[k][i];
        op(vi, oi);
#pragma unroll
        for (int k = 0; k < NOUT; ++k) o[k][i] = oi[k];
      }
#pragma unroll
      for (int k = 0; k < NOUT; ++k) st_pair<R>(out[k], t.rhs, t.p, j, wv, o[k]);
      j += 64;
      if (j < t.j1)
#pragma unroll
        for (int k = 0; k < NIN; ++k) ld_pair<R>(in[k], t.rhs, t.p, j, wv, v[k]);
    }
  }
}

template <class A> __device__ __forceinline__ double abs2(cx<A> v) {
  return (double)v.r * v.r + (double)v.i * v.i;
}

// reads the components of a tile of NIN fields into op(in)
template <class R, int NIN, class Op>
__device__ __forceinline__ void scan(const Tile& t, long long Vhp, const Field<R> (&in)[NIN], Op op) {
  typedef arith_t<R> A;
  if constexpr (is_h16<R>) {
    for (long long j = t.j0 + threadIdx.x; j < t.j1; j += BT<R>) {
      SiteR<R> r[NIN];
#pragma unroll
      for (int k = 0; k < NIN; ++k) r[k] = site_r(in[k], t.rhs, t.p, j, Vhp);
#pragma unroll
      for (int c = 0; c < 12; ++c) {
        cx<A> v[NIN];
#pragma unroll
        for (int k = 0; k < NIN; ++k) v[k] = get(r[k], c);
        op(v);
      }
    }
  } else {
    const int wv = threadIdx.x >> 6;
    for (long long j = t.j0 + (threadIdx.x & 63); j < t.j1; j += 64) {
      cx<A> v[NIN][2];
#pragma unroll
      for (int k = 0; k < NIN; ++k) ld_pair<R>(in[k], t.rhs, t.p, j, wv, v[k]);
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        cx<A> vi[NIN];
#pragma unroll
        for (int k = 0; k < NIN; ++k) vi[k] = v[k][i];
        op(vi);
      }
    }
  }
}

template <class R>
__global__ __launch_bounds__(BT<R>) void k_norm2(SysGrid G, Field<R> a, int npar, double* part) {
  __shared__ double sh[BT<R> / 64];
  const Tile t = tile_of(G, npar);
  double acc[1] = {0.0};
  if (t.selected) scan<R, 1>(t, G.Vhp, {a}, [&](const cx<arith_t<R>>* v) { acc[0] += abs2(v[0]); });
  block_sums<BT<R>, 1>(acc, sh);
  if (threadIdx.x == 0) part[t.part] = acc[0];
}

// ---- CG ---------------------------------------------------------------------------------

template <class R>
__global__ __launch_bounds__(BT<R>) void k_cg_s(SysGrid G, Field<R> s, Field<R> q, SysScal S, int v, Parts qq,
                                               double* part) {
  typedef arith_t<R> A;
  __shared__ double sh[2][BT<R> / 64];
  const Tile t = tile_of(G, 1, S.rev != 0);
  const double gam = S.gam[v * S.nsys + t.sys];
  const bool act = S.active[v * S.nsys + t.sys];
  if (S.nsys > 1 && !act) return;                                // whole workgroup
  double acc[1] = {0.0};
  A al = A(0);
  stream<R, 2, 1>(
      t, G.Vhp, {s, q}, {s},
      [&] {
        double n[1];
        thread_parts<BT<R>, 1>(qq, t.sys, n);
        block_sums<BT<R>, 1>(n, sh[0]);
        const double a = n[0] > 0.0 ? gam / n[0] : 0.0;
        al = (A)a;
        if (t.chunk == 0 && threadIdx.x == 0) {
          S.alpha[t.sys] = a;
          if (act && !isfinite(n[0])) S.flags[0] = 2;
        }
        return act;
      },
      [&](const cx<A>* in, cx<A>* out) {
        out[0] = {in[0].r - al * in[1].r, in[0].i - al * in[1].i};
        acc[0] += abs2(out[0]);
      });
  block_sums<BT<R>, 1>(acc, sh[1]);
  if (threadIdx.x == 0) part[t.part] = acc[0];
}

template <class R>
__global__ __launch_bounds__(BT<R>) void k_cg_xp(SysGrid G, Field<R> x, Field<R> p, Field<R> r, SysScal S, int v,
                                                Parts pss, Parts prr) {
  typedef arith_t<R> A;
  __shared__ double sh[2 * (BT<R> / 64)];
  const Tile t = tile_of(G, 1, S.rev != 0);
  const bool first = t.chunk == 0 && threadIdx.x == 0;
  const long long o = v * S.nsys + t.sys, n = (1 - v) * S.nsys + t.sys;
  const double gam = S.gam[o];
  const bool act = S.active[o];
  if (first && !act) {
    S.gam[n] = gam;
    S.active[n] = 0;
  }
  if (S.nsys > 1 && !act) return;                                // whole workgroup
  A al = (A)S.alpha[t.sys], be = A(0);
  stream<R, 3, 2>(
      t, G.Vhp, {x, p, r}, {x, p},
      [&] {
        if (!act) return false;
        double m[2];
        thread_parts<BT<R>, 1>(pss, t.sys, m);
        thread_parts<BT<R>, 1>(prr, t.sys, m + 1);
        block_sums<BT<R>, 2>(m, sh);
        be = (A)(gam > 0.0 ? m[1] / gam : 0.0);
        if (first) {
          if (!(isfinite(m[0]) && isfinite(m[1]))) S.flags[0] = 3;
          S.iters[t.sys] += 1;
          S.ss[t.sys] = m[0];
          S.gam[n] = m[1];
          S.active[n] = !(m[0] <= S.target2[t.sys] || m[1] == 0.0);
        }
        return true;
      },
      [&](const cx<A>* in, cx<A>* out) {
        out[0] = {in[0].r + al * in[1].r, in[0].i + al * in[1].i};
        out[1] = {in[2].r + be * in[1].r, in[2].i + be * in[1].i};
      });
}

// ---- precision changes and residuals ------------------------------------------------------

// out = scale * src on the even sites, converting precision, partial ||out||^2 (before any
// rounding to FP16); zero on unselected systems
template <class Ro>
__global__ __launch_bounds__(BT<Ro>) void k_convert(SysGrid G, Field<Ro> out, Field<double> in, double scale,
                                                   double* part) {
  typedef arith_t<Ro> Ao;
  __shared__ double sh[BT<Ro> / 64];
  const Tile t = tile_of(G);
  double acc[1] = {0.0};
  if constexpr (is_h16<Ro>) {
    for (long long j = t.j0 + threadIdx.x; j < t.j1; j += BT<Ro>) {
      const SiteR<double> ir = site_r(in, t.rhs, 0, j, G.Vhp);
      SiteW<Ro> ow = site_w(out, t.rhs, 0, j, G.Vhp);
#pragma unroll
      for (int c = 0; c < 12; ++c) {
        const cx<double> v = get(ir, c);
        cx<Ao> w = {(Ao)(scale * v.r), (Ao)(scale * v.i)};
        if (!t.selected) w = {Ao(0), Ao(0)};
        put(ow, c, w);
        acc[0] += abs2(w);
      }
      close(ow);
    }
  } else {
    const int wv = threadIdx.x >> 6;
    for (long long j = t.j0 + (threadIdx.x & 63); j < t.j1; j += 64) {
      cx<double> v[2];
      cx<Ro> w[2];
      ld_pair<double>(in, t.rhs, 0, j, wv, v);
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        w[i] = t.selected ? cx<Ro>{(Ro)(scale * v[i].r), (Ro)(scale * v[i].i)} : cx<Ro>{Ro(0), Ro(0)};
        acc[0] += abs2(w[i]);
      }
      st_pair<Ro>(out, t.rhs, 0, j, wv, w);
    }
  }
  block_sums<BT<Ro>, 1>(acc, sh);
  if (threadIdx.x == 0) part[t.part] = acc[0];
}

// even sites of the selected systems: x += e, e at the inner precision, and w = b - aI x
template <class R>
__global__ __launch_bounds__(BT<R>) void k_add_resid(SysGrid G, Field<double> x, Field<R> e, Field<double> b,
                                                    Field<double> w, double aI) {
  const Tile t = tile_of(G);
  if (!t.selected) return;
  if constexpr (is_h16<R>) {
    for (long long j = t.j0 + threadIdx.x; j < t.j1; j += BT<R>) {
      const SiteR<R> er = site_r(e, t.rhs, 0, j, G.Vhp);
#pragma unroll
      for (int c = 0; c < 12; ++c) {
        const long long o = tiled(j, c, 12);
        const cx<float> ev = get(er, c);
        cx<double> xv = ld<double>(x.ptr + t.rhs * x.rs + o);
        const cx<double> bv = ld<double>(b.ptr + t.rhs * b.rs + o);
        xv = {xv.r + (double)ev.r, xv.i + (double)ev.i};
        st<double>(x.ptr + t.rhs * x.rs + o, xv);
        st<double>(w.ptr + t.rhs * w.rs + o, {bv.r - aI * xv.r, bv.i - aI * xv.i});
      }
    }
  } else {
    const int wave = threadIdx.x >> 6;
    for (long long j = t.j0 + (threadIdx.x & 63); j < t.j1; j += 64) {
      cx<double> xv[2], bv[2], wv[2];
      cx<R> ev[2];
      ld_pair<double>(x, t.rhs, 0, j, wave, xv);
      ld_pair<double>(b, t.rhs, 0, j, wave, bv);
      ld_pair<R>(e, t.rhs, 0, j, wave, ev);
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        xv[i] = {xv[i].r + (double)ev[i].r, xv[i].i + (double)ev[i].i};
        wv[i] = {bv[i].r - aI * xv[i].r, bv[i].i - aI * xv[i].i};
      }
      st_pair<double>(x, t.rhs, 0, j, wave, xv);
      st_pair<double>(w, t.rhs, 0, j, wave, wv);
    }
  }
}

// ---- sums of partials outside the iterations: one workgroup, a wavefront per system ---------
constexpr int FT = 1024;

template <int N> __device__ __forceinline__ void wave_parts(Parts a, long long sys, double v[N]) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int k = 0; k < N; ++k) v[k] = 0.0;
  const double* q = a.p + sys * a.n * N;
  for (int i = lane; i < a.n; i += 64)
#pragma unroll
    for (int k = 0; k < N; ++k) v[k] += q[i * N + k];
#pragma unroll
  for (int k = 0; k < N; ++k) v[k] = wave_sum(v[k]);
}

// f(sys) by lane 0 of a wavefront for every system, after the N sums of its partials
template <int N, class F> __device__ __forceinline__ void each_system(int nsys, Parts a, F f) {
  for (int s = threadIdx.x >> 6; s < nsys; s += FT / 64) {
    double v[N];
    wave_parts<N>(a, s, v);
    if ((threadIdx.x & 63) == 0) f(s, v);
  }
}

__global__ __launch_bounds__(FT) void k_fin_sum(int nsys, Parts a, double* out) {
  each_system<1>(nsys, a, [&](int s, const double* v) { out[s] = v[0]; });
}

__global__ __launch_bounds__(FT) void k_fin_sum3(int nsys, Parts a, double* out) {
  each_system<3>(nsys, a, [&](int s, const double* v) {
    for (int k = 0; k < 3; ++k) out[3 * s + k] = v[k];
  });
}

__global__ __launch_bounds__(FT) void k_targets(int nsys, Parts bh, const double* bnorm2, double inner2, double abs2,
                                               double* target2) {
  each_system<1>(nsys, bh, [&](int s, const double* v) { target2[s] = fmax(inner2 * v[0], abs2 * bnorm2[s]); });
}

// sums of up to 256 neighbouring partials (nv values each): grid (groups, systems)
__global__ __launch_bounds__(256) void k_compress(int nv, Parts a, double* out) {
  __shared__ double sh[4];
  const int i = blockIdx.x * 256 + threadIdx.x;
  for (int k = 0; k < nv; ++k) {
    double v[1] = {i < a.n ? a.p[((long long)blockIdx.y * a.n + i) * nv + k] : 0.0};
    block_sums<256, 1>(v, sh);
    if (threadIdx.x == 0) out[((long long)blockIdx.y * gridDim.x + blockIdx.x) * nv + k] = v[0];
    __syncthreads();
  }
}

// Start of an inner CG: ||b_hat||^2, gam = ||r||^2; the system is active unless unselected
// or already below its target.
__global__ __launch_bounds__(FT) void k_fin_init(SysScal S, Parts b, Parts r) {
  __shared__ int cnt;
  if (threadIdx.x == 0) cnt = 0;
  __syncthreads();
  each_system<1>(S.nsys, b, [&](int s, const double* v) { S.ss[s] = v[0]; });
  __syncthreads();
  each_system<1>(S.nsys, r, [&](int s, const double* v) {
    const double bb = S.ss[s], gm = v[0];
    S.gam[s] = gm;
    S.alpha[s] = 0.0;
    const int act = S.selected[s] && bb > S.target2[s] && gm > 0.0;
    S.active[s] = act;
    if (!(isfinite(bb) && isfinite(gm))) S.flags[0] = 1;
    if (act) atomicAdd(&cnt, 1);
  });
  __syncthreads();
  if (threadIdx.x == 0) S.flags[1] = cnt;
}

__global__ __launch_bounds__(256) void k_fin_count(SysScal S, int v) {
  __shared__ double sh[4];
  double n[1] = {0.0};
  for (int s = threadIdx.x; s < S.nsys; s += 256) n[0] += S.active[v * S.nsys + s] ? 1.0 : 0.0;
  block_sums<256, 1>(n, sh);
  if (threadIdx.x == 0) S.flags[1] = (int)n[0];
}

// ---- BiCGstab -------------------------------------------------------------------------------

struct Cs {
  cx<double> rho, alpha, omega, beta;
};
__device__ __forceinline__ Cs cs_get(const SysScal& S, int v, long long sys) {
  const double* c = S.cs + 8 * (v * (long long)S.nsys + sys);
  return {{c[0], c[1]}, {c[2], c[3]}, {c[4], c[5]}, {c[6], c[7]}};
}
__device__ __forceinline__ void cs_set(const SysScal& S, int v, long long sys, const Cs& a) {
  double* c = S.cs + 8 * (v * (long long)S.nsys + sys);
  c[0] = a.rho.r; c[1] = a.rho.i; c[2] = a.alpha.r; c[3] = a.alpha.i;
  c[4] = a.omega.r; c[5] = a.omega.i; c[6] = a.beta.r; c[7] = a.beta.i;
}
__device__ __forceinline__ cx<double> cdiv(cx<double> a, cx<double> b) {
  const double d = b.r * b.r + b.i * b.i;
  return {(a.r * b.r + a.i * b.i) / d, (a.i * b.r - a.r * b.i) / d};
}

template <class R>
__global__ __launch_bounds__(BT<R>) void k_cdot3(SysGrid G, Field<R> a, Field<R> b, Field<R> c, double* part) {
  typedef arith_t<R> A;
  __shared__ double sh[3 * (BT<R> / 64)];
  const Tile t = tile_of(G);
  double s[3] = {0.0, 0.0, 0.0};
  auto dot = [&](const cx<A>& u, const cx<A>& v) {
    s[0] += (double)u.r * v.r + (double)u.i * v.i;
    s[1] += (double)u.r * v.i - (double)u.i * v.r;
  };
  if (t.selected) {
    if (c.ptr == nullptr)
      scan<R, 2>(t, G.Vhp, {a, b}, [&](const cx<A>* v) { dot(v[0], v[1]); });
    else if (c.ptr == a.ptr)
      scan<R, 2>(t, G.Vhp, {a, b}, [&](const cx<A>* v) { dot(v[0], v[1]); s[2] += abs2(v[0]); });
    else
      scan<R, 3>(t, G.Vhp, {a, b, c}, [&](const cx<A>* v) { dot(v[0], v[1]); s[2] += abs2(v[2]); });
  }
  block_sums<BT<R>, 3>(s, sh);
  if (threadIdx.x < 3) part[3 * t.part + threadIdx.x] = s[threadIdx.x];
}

// Close an iteration: rho_new = <r0, r>, stop on ||r||^2 <= target2, beta = (rho_new / rho)
// (alpha / omega). A breakdown (|<r0, r>|^2 <= 1e-24 ||r0||^2 ||r||^2, a zero rho or omega, or
// ||r|| > 1e6 ||r0||, beyond which FP32 iterates would overflow) stops the system, which the
// defect-correction loop then restarts from its current solution.
__device__ __forceinline__ bool rho_step(const double m[3], bool act, double gam, double target2, Cs& c) {
  const cx<double> rn = {m[0], m[1]};
  const double rr = m[2];
  act = act && rr > target2;
  const double rho2 = c.rho.r * c.rho.r + c.rho.i * c.rho.i, om2 = c.omega.r * c.omega.r + c.omega.i * c.omega.i;
  const double rn2 = rn.r * rn.r + rn.i * rn.i;
  if (act && (rho2 == 0.0 || om2 == 0.0 || !(rn2 > 1e-24 * gam * rr) || rr > 1e12 * gam)) act = false;
  if (act) {
    c.beta = cmul(cdiv(rn, c.rho), cdiv(c.alpha, c.omega));
    c.rho = rn;
  } else {
    c.beta = c.alpha = c.omega = {0.0, 0.0};
  }
  return act;
}

__global__ __launch_bounds__(FT) void k_fin_bicg_rho(SysScal S, int v, Parts a, int init) {
  __shared__ int cnt;
  if (threadIdx.x == 0) cnt = 0;
  __syncthreads();
  each_system<3>(S.nsys, a, [&](int s, const double* m) {
    if (!(isfinite(m[0]) && isfinite(m[1]) && isfinite(m[2]))) S.flags[0] = 4;
    const int w = init ? 0 : 1 - v;
    Cs c = {{1.0, 0.0}, {1.0, 0.0}, {1.0, 0.0}, {0.0, 0.0}};
    bool act = S.selected[s];
    if (init) {
      S.gam[s] = m[2];   // ||r0||^2 (r0 = r at the start)
    } else {
      c = cs_get(S, v, s);
      act = S.active[v * S.nsys + s];
    }
    act = rho_step(m, act, S.gam[s], S.target2[s], c);
    S.ss[s] = m[2];
    cs_set(S, w, s, c);
    S.active[w * S.nsys + s] = act;
    if (act) atomicAdd(&cnt, 1);
  });
  __syncthreads();
  if (threadIdx.x == 0) S.flags[1] = cnt;
}

template <class R>
__global__ __launch_bounds__(BT<R>) void k_bicg_p(SysGrid G, Field<R> p, Field<R> r, Field<R> vf, SysScal S, int v,
                                                 Parts rho) {
  typedef arith_t<R> A;
  __shared__ double sh[3 * (BT<R> / 64)];
  const Tile t = tile_of(G, 1, S.rev != 0);
  Cs c = cs_get(S, v, t.sys);
  bool act = S.active[v * S.nsys + t.sys];
  cx<A> b, w;
  stream<R, 3, 1>(
      t, G.Vhp, {p, r, vf}, {p},
      [&] {
        if (rho.p) {
          if (act) {
            double m[3];
            thread_parts<BT<R>, 3>(rho, t.sys, m);
            block_sums<BT<R>, 3>(m, sh);
            if (t.chunk == 0 && threadIdx.x == 0) {
              if (!(isfinite(m[0]) && isfinite(m[1]) && isfinite(m[2]))) S.flags[0] = 4;
              S.ss[t.sys] = m[2];
            }
            act = rho_step(m, act, S.gam[t.sys], S.target2[t.sys], c);
          }
          if (t.chunk == 0 && threadIdx.x == 0) {
            cs_set(S, 1 - v, t.sys, c);
            S.active[(1 - v) * S.nsys + t.sys] = act;
          }
        }
        b = {(A)c.beta.r, (A)c.beta.i};
        w = {(A)c.omega.r, (A)c.omega.i};
        return act;
      },
      [&](const cx<A>* in, cx<A>* out) { out[0] = in[1] + cmul(b, in[0] - cmul(w, in[2])); });
}

template <class R>
__global__ __launch_bounds__(BT<R>) void k_bicg_s(SysGrid G, Field<R> r, Field<R> vf, SysScal S, int v, Parts den,
                                                 double* part) {
  typedef arith_t<R> A;
  __shared__ double sh[2][3 * (BT<R> / 64)];
  const Tile t = tile_of(G, 1, S.rev != 0);
  Cs c = cs_get(S, v, t.sys);
  bool act = S.active[v * S.nsys + t.sys];
  double acc[1] = {0.0};
  cx<A> a = {A(0), A(0)};
  stream<R, 2, 1>(
      t, G.Vhp, {r, vf}, {r},
      [&] {
        if (act) {
          double m[3];
          thread_parts<BT<R>, 3>(den, t.sys, m);
          block_sums<BT<R>, 3>(m, sh[0]);
          if (t.chunk == 0 && threadIdx.x == 0 && !(isfinite(m[0]) && isfinite(m[1]))) S.flags[0] = 5;
          act = m[0] != 0.0 || m[1] != 0.0;
          c.alpha = act ? cdiv(c.rho, {m[0], m[1]}) : cx<double>{0.0, 0.0};
        }
        if (t.chunk == 0 && threadIdx.x == 0) {
          cs_set(S, 1 - v, t.sys, c);
          S.active[(1 - v) * S.nsys + t.sys] = act;
        }
        a = {(A)c.alpha.r, (A)c.alpha.i};
        return act;
      },
      [&](const cx<A>* in, cx<A>* out) {
        out[0] = in[0] - cmul(a, in[1]);
        acc[0] += abs2(out[0]);
      });
  block_sums<BT<R>, 1>(acc, sh[1]);
  if (threadIdx.x == 0) part[t.part] = acc[0];
}

// omega = <t, s> / ||t||^2. When ||s||^2 already meets the target the step ends with
// x += alpha p (omega = 0, r = s); when <t, s> (nearly) vanishes the system stops after
// that same update (breakdown, restarted by the defect-correction loop).
template <class R>
__global__ __launch_bounds__(BT<R>) void k_bicg_xr(SysGrid G, Field<R> x, Field<R> p, Field<R> r, Field<R> tt,
                                                  Field<R> r0, SysScal S, int v, Parts ts, Parts pss, double* part) {
  typedef arith_t<R> A;
  __shared__ double sh[2][4 * (BT<R> / 64)];
  const Tile t = tile_of(G, 1, S.rev != 0);
  const bool first = t.chunk == 0 && threadIdx.x == 0;
  Cs c = cs_get(S, v, t.sys);
  const bool act = S.active[v * S.nsys + t.sys];
  double acc[3] = {0.0, 0.0, 0.0};
  cx<A> a = {A(0), A(0)}, w = {A(0), A(0)};
  stream<R, 5, 2>(
      t, G.Vhp, {x, p, r, tt, r0}, {x, r},
      [&] {
        bool next = act;
        if (act) {
          double m[4];
          thread_parts<BT<R>, 3>(ts, t.sys, m);
          thread_parts<BT<R>, 1>(pss, t.sys, m + 3);
          block_sums<BT<R>, 4>(m, sh[0]);
          if (first) {
            if (!(isfinite(m[0]) && isfinite(m[1]) && isfinite(m[2]) && isfinite(m[3]))) S.flags[0] = 6;
            S.iters[t.sys] += 1;
          }
          c.omega = {0.0, 0.0};
          const double ts2 = m[0] * m[0] + m[1] * m[1];
          if (m[3] <= S.target2[t.sys]) {
            // converged on s: omega stays 0
          } else if (m[2] > 0.0 && ts2 > 1e-24 * m[2] * m[3]) {
            c.omega = {m[0] / m[2], m[1] / m[2]};
          } else {
            next = false;
          }
        }
        if (first) {
          cs_set(S, 1 - v, t.sys, c);
          S.active[(1 - v) * S.nsys + t.sys] = next;
        }
        a = {(A)c.alpha.r, (A)c.alpha.i};
        w = {(A)c.omega.r, (A)c.omega.i};
        return act;
      },
      [&](const cx<A>* in, cx<A>* out) {
        out[0] = in[0] + cmul(a, in[1]) + cmul(w, in[2]);
        const cx<A> rn = in[2] - cmul(w, in[3]), q = in[4];
        out[1] = rn;
        acc[0] += (double)q.r * rn.r + (double)q.i * rn.i;
        acc[1] += (double)q.r * rn.i - (double)q.i * rn.r;
        acc[2] += abs2(rn);
      });
  block_sums<BT<R>, 3>(acc, sh[1]);
  if (threadIdx.x < 3) part[3 * t.part + threadIdx.x] = acc[threadIdx.x];
}

template <class R>
__global__ __launch_bounds__(BT<R>) void k_lin3(SysGrid G, Field<R> y, Field<R> u, Field<R> w, Field<R> q,
                                              const double* coef, double* part) {
  typedef arith_t<R> A;
  __shared__ double sh[3 * (BT<R> / 64)];
  const Tile t = tile_of(G);
  double s[3] = {0.0, 0.0, 0.0};
  if (t.selected) {
    const double* cf = coef + 6 * t.sys;
    const cx<A> c0 = {(A)cf[0], (A)cf[1]}, c1 = {(A)cf[2], (A)cf[3]}, c2 = {(A)cf[4], (A)cf[5]};
    const bool keep_y = cf[0] != 0.0 || cf[1] != 0.0;   // c0 = 0: y is not read (may be unset)
    const bool with_w = w.ptr != nullptr, with_q = q.ptr != nullptr;
    const int wv = threadIdx.x >> 6;
    for (long long j = t.j0 + (threadIdx.x & 63); j < t.j1; j += 64) {
      cx<A> uv[2], yv[2], ww[2], qv[2], o[2];
      ld_pair<R>(u, t.rhs, t.p, j, wv, uv);
      if (keep_y) ld_pair<R>(y, t.rhs, t.p, j, wv, yv);
      if (with_w) ld_pair<R>(w, t.rhs, t.p, j, wv, ww);
      if (with_q) ld_pair<R>(q, t.rhs, t.p, j, wv, qv);
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        cx<A> v = cmul(c1, uv[i]);
        if (keep_y) v = v + cmul(c0, yv[i]);
        if (with_w) v = v + cmul(c2, ww[i]);
        o[i] = v;
        if (with_q) {
          s[0] += (double)qv[i].r * v.r + (double)qv[i].i * v.i;
          s[1] += (double)qv[i].r * v.i - (double)qv[i].i * v.r;
        }
        s[2] += abs2(v);
      }
      st_pair<R>(y, t.rhs, t.p, j, wv, o);
    }
  }
  if (part) {
    block_sums<BT<R>, 3>(s, sh);
    if (threadIdx.x < 3) part[3 * t.part + threadIdx.x] = s[threadIdx.x];
  }
}

// ---- geometric series -----------------------------------------------------------------------

// A system stops once the new term satisfies ||t||^2 <= target2, and is flagged divergent
// once ||t||^2 > 1e30 ||b_hat||^2 (ss keeps ||t_0||^2 = ||b_hat||^2).
__device__ __forceinline__ bool geom_step(const SysScal& S, long long sys, double tt, bool record) {
  if (record && !isfinite(tt)) S.flags[0] = 7;
  if (record) S.iters[sys] += 1;
  if (tt <= S.target2[sys]) return false;
  if (!(tt <= 1e30 * S.ss[sys])) {
    if (record) S.flags[2] = 1;
    return false;
  }
  return true;
}

__global__ __launch_bounds__(FT) void k_fin_geom(SysScal S, int v, Parts a, int init) {
  __shared__ int cnt;
  if (threadIdx.x == 0) cnt = 0;
  __syncthreads();
  each_system<1>(S.nsys, a, [&](int s, const double* m) {
    bool act;
    if (init) {
      if (!isfinite(m[0])) S.flags[0] = 7;
      act = S.selected[s] && m[0] > S.target2[s];
      S.ss[s] = m[0];
    } else {
      act = S.active[v * S.nsys + s] && geom_step(S, s, m[0], true);
    }
    S.active[(init ? 0 : 1 - v) * S.nsys + s] = act;
    if (act) atomicAdd(&cnt, 1);
  });
  __syncthreads();
  if (threadIdx.x == 0) S.flags[1] = cnt;
}

template <class R>
__global__ __launch_bounds__(BT<R>) void k_geom_add(SysGrid G, Field<R> x, Field<R> tf, SysScal S, int v, Parts tt) {
  typedef arith_t<R> A;
  __shared__ double sh[BT<R> / 64];
  const Tile t = tile_of(G, 1, S.rev != 0);
  bool act = S.active[v * S.nsys + t.sys];
  stream<R, 2, 1>(
      t, G.Vhp, {x, tf}, {x},
      [&] {
        if (tt.p) {
          const bool first = t.chunk == 0 && threadIdx.x == 0;
          if (act) {
            double m[1];
            thread_parts<BT<R>, 1>(tt, t.sys, m);
            block_sums<BT<R>, 1>(m, sh);
            act = geom_step(S, t.sys, m[0], first);
          }
          if (first) S.active[(1 - v) * S.nsys + t.sys] = act;
        }
        return act;
      },
      [&](const cx<A>* in, cx<A>* out) { out[0] = in[0] + in[1]; });
}

inline dim3 grid_of(const SysGrid& G, int nrhs, int npar = 1) {
  return G.xcd ? dim3(G.nchunk * G.nblk * nrhs * npar) : dim3(G.nchunk, G.nblk, nrhs * npar);
}

}  // namespace

// ---------------------------------------------------------------------------------
template <class R> void blas_norm2(const SysGrid& G, int nrhs, Field<R> a, int npar, double* part, hipStream_t s) {
  hipLaunchKernelGGL(k_norm2<R>, grid_of(G, nrhs, npar), dim3(BT<R>), 0, s, G, a, npar, part);
}
template <class R> void blas_cg_s(const SysGrid& G, int nrhs, Field<R> sf, Field<R> q, const SysScal& S, int v,
                                  Parts qq, double* part, hipStream_t s) {
  hipLaunchKernelGGL(k_cg_s<R>, grid_of(G, nrhs), dim3(BT<R>), 0, s, G, sf, q, S, v, qq, part);
}
template <class R> void blas_cg_xp(const SysGrid& G, int nrhs, Field<R> x, Field<R> p, Field<R> r, const SysScal& S,
                                   int v, Parts ss, Parts rr, hipStream_t s) {
  hipLaunchKernelGGL(k_cg_xp<R>, grid_of(G, nrhs), dim3(BT<R>), 0, s, G, x, p, r, S, v, ss, rr);
}
template <class R> void blas_convert(const SysGrid& G, int nrhs, Field<R> out, Field<double> in, double scale,
                                     double* part, hipStream_t s) {
  hipLaunchKernelGGL(k_convert<R>, grid_of(G, nrhs), dim3(BT<R>), 0, s, G, out, in, scale, part);
}
template <class R> void blas_add_resid(const SysGrid& G, int nrhs, Field<double> x, Field<R> e, Field<double> b,
                                       Field<double> w, double aI, hipStream_t s) {
  hipLaunchKernelGGL(k_add_resid<R>, grid_of(G, nrhs), dim3(BT<R>), 0, s, G, x, e, b, w, aI);
}
void fin_sum(int nsys, Parts a, double* out, hipStream_t s) {
  hipLaunchKernelGGL(k_fin_sum, dim3(1), dim3(FT), 0, s, nsys, a, out);
}
void fin_sum3(int nsys, Parts a, double* out, hipStream_t s) {
  hipLaunchKernelGGL(k_fin_sum3, dim3(1), dim3(FT), 0, s, nsys, a, out);
}
void fin_targets(int nsys, Parts bh, const double* bnorm2, double inner2, double abs2, double* target2,
                 hipStream_t s) {
  hipLaunchKernelGGL(k_targets, dim3(1), dim3(FT), 0, s, nsys, bh, bnorm2, inner2, abs2, target2);
}
int compress_parts(int nsys, int nv, Parts a, double* out, hipStream_t s) {
  const int n = (a.n + 255) / 256;
  hipLaunchKernelGGL(k_compress, dim3(n, nsys), dim3(256), 0, s, nv, a, out);
  return n;
}
void fin_init(const SysScal& S, Parts b, Parts r, hipStream_t s) {
  hipLaunchKernelGGL(k_fin_init, dim3(1), dim3(FT), 0, s, S, b, r);
}
void fin_count(const SysScal& S, int v, hipStream_t s) {
  hipLaunchKernelGGL(k_fin_count, dim3(1), dim3(256), 0, s, S, v);
}
template <class R> void blas_cdot3(const SysGrid& G, int nrhs, Field<R> a, Field<R> b, Field<R> c, double* part,
                                   hipStream_t s) {
  hipLaunchKernelGGL(k_cdot3<R>, grid_of(G, nrhs), dim3(BT<R>), 0, s, G, a, b, c, part);
}
template <class R> void blas_bicg_p(const SysGrid& G, int nrhs, Field<R> p, Field<R> r, Field<R> v, const SysScal& S,
                                    int ver, Parts rho, hipStream_t s) {
  hipLaunchKernelGGL(k_bicg_p<R>, grid_of(G, nrhs), dim3(BT<R>), 0, s, G, p, r, v, S, ver, rho);
}
template <class R> void blas_bicg_s(const SysGrid& G, int nrhs, Field<R> r, Field<R> v, const SysScal& S, int ver,
                                    Parts den, double* part, hipStream_t s) {
  hipLaunchKernelGGL(k_bicg_s<R>, grid_of(G, nrhs), dim3(BT<R>), 0, s, G, r, v, S, ver, den, part);
}
template <class R> void blas_bicg_xr(const SysGrid& G, int nrhs, Field<R> x, Field<R> p, Field<R> r,
                                     Field<R> t, Field<R> r0, const SysScal& S, int ver, Parts ts, Parts ss,
                                     double* part, hipStream_t s) {
  hipLaunchKernelGGL(k_bicg_xr<R>, grid_of(G, nrhs), dim3(BT<R>), 0, s, G, x, p, r, t, r0, S, ver, ts, ss, part);
}
void fin_bicg_rho(const SysScal& S, int ver, Parts a, int init, hipStream_t s) {
  hipLaunchKernelGGL(k_fin_bicg_rho, dim3(1), dim3(FT), 0, s, S, ver, a, init);
}
template <class R> void blas_geom_add(const SysGrid& G, int nrhs, Field<R> x, Field<R> t, const SysScal& S, int ver,
                                      Parts tt, hipStream_t s) {
  hipLaunchKernelGGL(k_geom_add<R>, grid_of(G, nrhs), dim3(BT<R>), 0, s, G, x, t, S, ver, tt);
}
void fin_geom(const SysScal& S, int ver, Parts tt, int init, hipStream_t s) {
  hipLaunchKernelGGL(k_fin_geom, dim3(1), dim3(FT), 0, s, S, ver, tt, init);
}
template <class R> void blas_lin3(const SysGrid& G, int nrhs, Field<R> y, Field<R> u, Field<R> w, Field<R> q,
                                  const double* coef, double* part, hipStream_t s) {
  hipLaunchKernelGGL(k_lin3<R>, grid_of(G, nrhs), dim3(BT<R>), 0, s, G, y, u, w, q, coef, part);
}

#define INST(R)                                                                                              \
  template void blas_norm2<R>(const SysGrid&, int, Field<R>, int, double*, hipStream_t);                      \
  template void blas_cg_s<R>(const SysGrid&, int, Field<R>, Field<R>, const SysScal&, int, Parts, double*,    \
                             hipStream_t);                                                                    \
  template void blas_cg_xp<R>(const SysGrid&, int, Field<R>, Field<R>, Field<R>, const SysScal&, int, Parts,  \
                              Parts, hipStream_t);                                                            \
  template void blas_convert<R>(const SysGrid&, int, Field<R>, Field<double>, double, double*, hipStream_t);  \
  template void blas_add_resid<R>(const SysGrid&, int, Field<double>, Field<R>, Field<double>, Field<double>, \
                                  double, hipStream_t);                                                       \
  template void blas_cdot3<R>(const SysGrid&, int, Field<R>, Field<R>, Field<R>, double*, hipStream_t);       \
  template void blas_bicg_p<R>(const SysGrid&, int, Field<R>, Field<R>, Field<R>, const SysScal&, int, Parts, \
                               hipStream_t);                                                                  \
  template void blas_bicg_s<R>(const SysGrid&, int, Field<R>, Field<R>, const SysScal&, int, Parts, double*,  \
                               hipStream_t);                                                                  \
  template void blas_bicg_xr<R>(const SysGrid&, int, Field<R>, Field<R>, Field<R>, Field<R>, Field<R>,        \
                                const SysScal&, int, Parts, Parts, double*, hipStream_t);                     \
  template void blas_geom_add<R>(const SysGrid&, int, Field<R>, Field<R>, const SysScal&, int, Parts, hipStream_t);
INST(double)
INST(float)
INST(h16)
template void blas_lin3<double>(const SysGrid&, int, Field<double>, Field<double>, Field<double>, Field<double>,
                                const double*, double*, hipStream_t);

}  // namespace sap
