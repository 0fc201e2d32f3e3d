// Batched Krylov solves of M x = b (full lattice) and W x = b (every selected x0 block
// an independent system), all systems and right-hand sides advanced together in each
// kernel launch.
//
// Inner solve: even-odd reduced system (Sec. 1, W_eo: M = [[1, -k D_eo], [-k D_oe, 1]],
// M_hat = 1 - k^2 D_eo D_oe), by one of
//  * CG on the normal equations in the CGLS form, which carries s = b_hat - M_hat x;
//    M_hat^dagger = g5 M_hat g5 is applied by the same hop kernel with gamma_5 folded
//    into its input and output;
//  * BiCGstab (van der Vorst) on M_hat directly, with complex per-system scalars;
//  * the geometric series x_e = sum_n (k^2 D_eo D_oe)^n b_hat (Sec. 3 uses it for the block
//    terms), whose residual after n terms is the next term; for the shifted even-site
//    system (M_hat + rho) x_e = b_e of the mass-preconditioned parts every term carries a
//    factor 1 / (1 + rho) and the residual after n terms is (1 + rho) times the next term.
// Per-system scalars stay on the device, formed by the kernels that need them from the
// partial sums (blas.hip), so that a CG iteration is six launches with the norms written by
// the hops; converged systems are frozen while the others continue; the host reads one
// counter every few iterations. On 16^3x32 with one rhs and FP32 inner iterations an
// iteration went from 93 us in ten launches to 52 us.
// Outer loop: FP64 defect correction on the even sites: r_e = b_hat - M_hat x_e in FP64, inner
// solve in FP16, FP32 or FP64, x_e += e, x_o = b_o + k D_oe x_e, until ||b - A x|| / ||b|| <=
// tol recomputed in FP64.
#include <algorithm>
#include <cmath>
#include <complex>
#include <cstring>
#include <vector>
#include "blas.h"
#include "split.h"

using namespace sap;

namespace sap {
int apply_op_any(sap_ctx* ctx, void* out, const void* in, int nrhs, int lb, int colour, int block,
                 sap_prec prec, hipStream_t s);
}

struct SolverWS {
  int max_rhs, max_sys;
  size_t part_cap;                       // doubles in each of partA ... partE
  double2 *hx, *s, *r, *p, *q, *t, *e;   // half fields (sized for FP64, max_rhs)
  double2 *r64, *ax;                     // full fields
  double *partA, *partB, *partC, *partD, *partE;
  double *gam, *ss, *alpha, *target2, *bnorm2, *rnorm2;
  double* cs;                            // BiCGstab: complex (rho, alpha, omega, beta) per system
                                         // (gam, cs and active: two versions)
  int *active, *iters, *flags, *selected;
  // pinned host mirrors
  double *h_rnorm2, *h_bnorm2;            // h_bnorm2: then ||b||^2 of each parity, two per system
  int *h_flags, *h_iters, *h_selected;
  // captured inner-loop graphs (ITERS_PER_GRAPH CG iterations each), replayed on the
  // caller's stream; captured on a private non-blocking stream of default priority
  hipStream_t cap;
  struct G { int nrhs, lb, sel, prec, method; double rho; hipGraphExec_t exec; };
  std::vector<G> graphs;
};

constexpr int ITERS_PER_GRAPH = 8;

static SolverWS* ws_of(sap_ctx* c) { return (SolverWS*)c->solver; }
struct SapWS;
static SapWS* sap_ws(sap_ctx* c);   // Schwarz-preconditioned BiCGstab workspace (below)

extern "C" int sap_solver_create(sap_ctx* c) {
  SolverWS* w = new SolverWS();   // value-initialised: every pointer starts null
  c->solver = w;
  const int minlb = c->geom.l0_sub > 0 ? c->geom.l0_sub : c->geom.l0;
  w->max_rhs = c->geom.max_rhs;
  w->max_sys = (c->geom.L[0] / minlb) * w->max_rhs;
  if (w->max_sys < w->max_rhs) w->max_sys = w->max_rhs;
  const size_t half = (size_t)12 * c->Vhp * w->max_rhs * sizeof(double2);
  const size_t full = 2 * half;
  // three partials per (system, 64-site chunk of each parity, the chunks of a block or of a
  // slice rounded up), or per slot of the LDS-staged hops
  size_t npart = 0;
  for (int nlb : {c->geom.l0, c->geom.l0_sub, c->geom.L[0]})
    if (nlb > 0) {
      const int per_sys = std::max(2 * split_chunks(c->g, nlb, true), slabd_norm_slots(c->g, nlb));
      npart = std::max(npart, (size_t)3 * w->max_rhs * (c->geom.L[0] / nlb) * per_sys);
    }
  w->part_cap = npart;
  auto A = [&](void** p, size_t n) { return hipMalloc(p, n) == hipSuccess; };
  bool ok = A((void**)&w->hx, half) && A((void**)&w->s, half) && A((void**)&w->r, half) &&
            A((void**)&w->p, half) && A((void**)&w->q, half) && A((void**)&w->t, half) &&
            A((void**)&w->e, half) && A((void**)&w->r64, full) && A((void**)&w->ax, full) &&
            A((void**)&w->partA, npart * 8) && A((void**)&w->partB, npart * 8) &&
            A((void**)&w->partC, npart * 8) && A((void**)&w->partD, npart * 8) &&
            A((void**)&w->partE, npart * 8);
  const size_t ns = (size_t)w->max_sys;
  ok = ok && A((void**)&w->gam, 2 * ns * 8) && A((void**)&w->ss, ns * 8) && A((void**)&w->alpha, ns * 8) &&
       A((void**)&w->target2, ns * 8) && A((void**)&w->bnorm2, ns * 8) &&
       A((void**)&w->rnorm2, ns * 8) && A((void**)&w->cs, 2 * ns * 64) && A((void**)&w->active, 2 * ns * 4) &&
       A((void**)&w->iters, ns * 4) &&
       A((void**)&w->flags, 16) && A((void**)&w->selected, ns * 4);
  ok = ok && hipHostMalloc((void**)&w->h_rnorm2, ns * 8, 0) == hipSuccess &&
       hipHostMalloc((void**)&w->h_bnorm2, 3 * ns * 8, 0) == hipSuccess &&
       hipHostMalloc((void**)&w->h_flags, 16, 0) == hipSuccess &&
       hipHostMalloc((void**)&w->h_iters, ns * 4, 0) == hipSuccess &&
       hipHostMalloc((void**)&w->h_selected, ns * 4, 0) == hipSuccess;
  if (!ok) return sap_fail(c, SAP_E_NOMEM, "cannot allocate the solver workspace");
  if (hipStreamCreateWithFlags(&w->cap, hipStreamNonBlocking) != hipSuccess)
    return sap_fail(c, SAP_E_HIP, "cannot create the capture stream");
  // the Schwarz-preconditioned BiCGstab workspace too, so that no solve allocates fields
  if (!sap_ws(c)) return sap_fail(c, SAP_E_NOMEM, "cannot allocate the Schwarz-preconditioned BiCGstab workspace");
  return SAP_OK;
}

static void drop_graphs(SolverWS* w) {
  for (auto& g : w->graphs) (void)hipGraphExecDestroy(g.exec);
  w->graphs.clear();
}

extern "C" void sap_solver_destroy(sap_ctx* c) {
  SolverWS* w = ws_of(c);
  if (!w) return;
  void* dev[] = {w->hx, w->s, w->r, w->p, w->q, w->t, w->e, w->r64, w->ax,
                 w->partA, w->partB, w->partC, w->partD, w->partE, w->gam, w->ss, w->alpha, w->target2,
                 w->bnorm2, w->rnorm2, w->cs, w->active, w->iters, w->flags, w->selected};
  for (void* p : dev)
    if (p) (void)hipFree(p);
  void* host[] = {w->h_rnorm2, w->h_bnorm2, w->h_flags, w->h_iters, w->h_selected};
  for (void* p : host)
    if (p) (void)hipHostFree(p);
  drop_graphs(w);
  if (w->cap) (void)hipStreamDestroy(w->cap);
  delete w;
  c->solver = nullptr;
}

namespace {

// reductions a half hop adds to its output for systems of nlb slices (HopArgs::npart)
struct Fused {
  double* part = nullptr;
  int nlb = 0, nslot = 0, red = 0;
  const int* active = nullptr;
  int keep = 0, rev = 0;
};

// out = a*x + b*D(in) on one parity or both, block-restricted
template <class R>
HopArgs<R> hop_args(sap_ctx* c, Field<R> out, Field<R> in, Field<R> x, int parity_out, int nrhs, int lb, int colour,
                    typename arith<R>::type a, typename arith<R>::type b, int g5i, int g5o) {
  HopArgs<R> A;
  A.out = out;
  A.in = in;
  A.x = x;
  A.U = gauge_of<R>(c);
  A.g = c->g;
  A.nrhs = nrhs;
  A.parity_out = parity_out;
  A.lb = lb;
  A.slb = lb;
  A.colour = colour < 3 ? colour : 0;
  A.block = colour < 3 ? -1 : colour - 3;
  A.a = a;
  A.b = b;
  A.g5_in = g5i;
  A.g5_out = g5o;
  A.map = hop_map_for(c, parity_out < 0, prec_of<R>(), nrhs,
                      parity_out < 0 ? hop_use(A.g, lb, A.colour, A.block) : (int)HOP_SOLVE);
  return A;
}
template <class R>
void hop(sap_ctx* c, Field<R> out, Field<R> in, Field<R> x, int parity_out, int nrhs, int lb, int colour,
         typename arith<R>::type a, typename arith<R>::type b, int g5i, int g5o, hipStream_t st, Fused f = {}) {
  HopArgs<R> A = hop_args<R>(c, out, in, x, parity_out, nrhs, lb, colour, a, b, g5i, g5o);
  A.npart = f.part;
  A.nlb = f.nlb;
  A.nslot = f.nslot;
  A.red = f.red;
  A.active = f.active;
  A.keep = f.keep;
  A.rev = f.rev;
  launch_hop<R>(A, st);
}

}  // namespace

template <class R>
// eo_only: solve (M_hat + rho) x_e = b_e on the even sites (x and b vanish on the odd
// sites; no reconstruction; residual on the even sites), the form the mass-preconditioned
// action parts need. Otherwise rho must be 0.
static int solve_impl(sap_ctx* c, double* x, const double* b, int nrhs, int lb, int colour,
                      const sap_solve_opts* o, sap_solve_info* info, hipStream_t st, double rho = 0.0,
                      bool eo_only = false) {
  typedef typename arith<R>::type Ar;
  SolverWS* w = ws_of(c);
  const long long Vh = c->Vh, Vhp = c->Vhp;
  const bool ranges = hop_in_ranges(hop_args<R>(c, {}, {}, {}, 0, nrhs, lb, colour, Ar(1), Ar(1), 0, 0));
  const SysGrid G = make_sysgrid(Vh, c->g.V3h, lb, c->geom.L[0], colour, nrhs, std::is_same<R, h16>::value, ranges);
  const int nsys = G.nblk * nrhs;
  const double kap = c->geom.kappa;
  const Ar k2R = (Ar)(-kap * kap);
  const Ar aI = (Ar)(1.0 + rho);               // unit term of M_hat + rho
  const size_t fullb = (size_t)24 * Vhp * nrhs * sizeof(double2), halfR = half_bytes<R>(Vhp, nrhs);
  if (rho != 0.0 && !eo_only) return sap_fail(c, SAP_E_ARG, "a shift needs the even-site system");
  // geometric series: terms t_0 = b_hat / (1 + rho), t_{n+1} = k^2 / (1 + rho) D_eo D_oe t_n,
  // residual (1 + rho) t_{n+1}: the series works on t, so b_hat and the target are scaled
  const bool geom = o->method == SAP_GEOM;
  const double shift_inv = 1.0 / (1.0 + rho);

  Field<double> X = {(double2*)x, 24 * Vhp, 12 * Vhp}, B = {(double2*)b, 24 * Vhp, 12 * Vhp};
  Field<double> R64 = {w->r64, 24 * Vhp, 12 * Vhp}, AX = {w->ax, 24 * Vhp, 12 * Vhp};
  Field<R> Ee = half_field<R>(w->e, Vhp);
  Field<R> S = half_field<R>(w->s, Vhp), Rr = half_field<R>(w->r, Vhp), P = half_field<R>(w->p, Vhp);
  Field<R> Q = half_field<R>(w->q, Vhp), T = half_field<R>(w->t, Vhp);
  Field<R> HX = half_field<R>(w->hx, Vhp);
  const int method = (int)o->method;
  Field<R> NONE = {nullptr, 0, 0, 0};
  const SysScal SC = {w->gam, w->ss, w->alpha, w->cs, w->active, w->iters, w->flags, w->selected, w->target2, nsys};
  const int n1 = G.nchunk, n2 = 2 * G.nchunk;   // partials per system of sums over one / both parities

  // selection of systems
  for (int r = 0; r < nrhs; ++r)
    for (int k = 0; k < G.nblk; ++k)
      w->h_selected[r * G.nblk + k] = block_selected(G.colour, k);
  SAP_HIP_CHECK(c, hipMemcpyAsync(w->selected, w->h_selected, nsys * 4, hipMemcpyHostToDevice, st));
  SAP_HIP_CHECK(c, hipMemsetAsync(w->iters, 0, nsys * 4, st));
  SAP_HIP_CHECK(c, hipMemsetAsync(x, 0, fullb, st));

  // ||b||^2 per system (the first residual), of even-site systems also by parity
  blas_norm2<double>(G, nrhs, B, 2, w->partA, st);
  fin_sum(nsys, {w->partA, n2}, w->bnorm2, st);
  SAP_HIP_CHECK(c, hipMemcpyAsync(w->h_bnorm2, w->bnorm2, nsys * 8, hipMemcpyDeviceToHost, st));
  double* const par2 = w->h_bnorm2 + w->max_sys;
  if (eo_only) {
    fin_sum(2 * nsys, {w->partA, n1}, w->gam, st);
    SAP_HIP_CHECK(c, hipMemcpyAsync(par2, w->gam, 2 * nsys * 8, hipMemcpyDeviceToHost, st));
  }

  const double tol = o->tol;
  const double inner_tol = (std::is_same<R, double>::value && o->inner_tol <= 0) ? tol : o->inner_tol;
  long long total_iters = 0;
  int outer = 0;
  int status = SAP_OK;
  for (;;) {
    if (outer) SAP_HIP_CHECK(c, hipMemcpyAsync(w->h_rnorm2, w->rnorm2, nsys * 8, hipMemcpyDeviceToHost, st));
    SAP_HIP_CHECK(c, hipStreamSynchronize(st));
    bool all = true, finite = true;
    for (int s = 0; s < nsys; ++s) {
      // (a source of the even-site system that does not vanish on the odd sites has no solution)
      if (!outer) w->h_rnorm2[s] = w->h_bnorm2[s];
      else if (eo_only) w->h_rnorm2[s] += par2[2 * s + 1];
      if (!w->h_selected[s]) continue;
      const double bb = w->h_bnorm2[s], rr = w->h_rnorm2[s];
      if (!std::isfinite(rr) || !std::isfinite(bb)) finite = false;
      if (bb > 0 && rr > tol * tol * bb) all = false;
    }
    if (!finite) { status = sap_fail(c, SAP_E_NONFINITE, "non-finite residual"); break; }
    if (all) break;
    if (outer >= o->max_outer || total_iters >= o->max_iter) {
      status = sap_fail(c, SAP_E_NOCONV, "solver did not reach tol within max_outer / max_iter");
      break;
    }
    ++outer;
    // the even-site residual of x = 0: b_hat = b_e + k D_eo b_o
    if (outer == 1 && !eo_only) hop<double>(c, R64, B, B, 0, nrhs, lb, colour, 1.0, kap, 0, 0, st);
    // inner right-hand side, the even-site residual at the inner precision (into S; times
    // 1 / (1 + rho) for the series)
    blas_convert<R>(G, nrhs, S, outer == 1 && eo_only ? B : R64, geom ? shift_inv : 1.0, w->partB, st);
    SAP_HIP_CHECK(c, hipMemsetAsync(w->e, 0, halfR, st));
    // stop the inner solve at ||s|| <= max(inner_tol ||b_hat||, 0.3 tol ||b||): the outer
    // residual after x += e equals the inner one up to rounding
    fin_targets(nsys, {w->partB, n1}, w->bnorm2, inner_tol * inner_tol,
                0.09 * tol * tol * (geom ? shift_inv * shift_inv : 1.0), w->target2, st);
    SAP_HIP_CHECK(c, hipMemsetAsync(w->flags, 0, 16, st));
    const size_t halfb = halfR;
    if (method == SAP_CG) {
      // r = M_hat^dagger s = s - k^2 g5 D_eo D_oe g5 s
      hop<R>(c, T, S, NONE, 1, nrhs, lb, colour, Ar(0), Ar(1), 1, 0, st);
      hop<R>(c, Rr, T, S, 0, nrhs, lb, colour, aI, k2R, 0, 1, st);
      blas_norm2<R>(G, nrhs, Rr, 1, w->partC, st);
      fin_init(SC, {w->partB, n1}, {w->partC, n1}, st);
      SAP_HIP_CHECK(c, hipMemcpyAsync(w->p, w->r, halfb, hipMemcpyDeviceToDevice, st));
    } else if (method == SAP_BICGSTAB) {
      // r = s = b_hat (x_e = 0), shadow residual r0 = r, p = v = 0
      SAP_HIP_CHECK(c, hipMemcpyAsync(w->r, w->s, halfb, hipMemcpyDeviceToDevice, st));
      SAP_HIP_CHECK(c, hipMemsetAsync(w->p, 0, halfb, st));
      SAP_HIP_CHECK(c, hipMemsetAsync(w->q, 0, halfb, st));
      blas_cdot3<R>(G, nrhs, Rr, S, S, w->partA, st);
      fin_bicg_rho(SC, 0, {w->partA, n1}, 1, st);
    } else {
      // first term t_0 = b_hat in S
      fin_geom(SC, 0, {w->partB, n1}, 1, st);
    }
    SAP_HIP_CHECK(c, hipGetLastError());
    // where its mapping can, the second half hop writes the reductions of its output: ||M_hat
    // p||^2 and ||M_hat^dagger s||^2 (CG), <t, s> and ||t||^2 (BiCGstab, three values per slot),
    // ||t||^2 (series); FP16 sums the values before their rounding to FP16
    const int nlb = lb ? lb : c->geom.L[0];
    int nslot = hop_red_slots(hop_args<R>(c, Q, T, P, 0, nrhs, lb, colour, aI, k2R, 0, 0), nlb);
    if ((size_t)3 * nslot * nsys > w->part_cap) nslot = 0;       // no room in the partial buffers
    // the updates skip converged systems (version v of active), also a single one, and so do the
    // hops of the mappings that HopArgs::active names: a graph runs up to seven iterations past
    // its end. Separate norm and dot passes run for every selected system.
    auto live = [&](int v) { return w->active + v * nsys; };
    // consecutive kernels walk the lattice in opposite directions, so that each begins with
    // what the one before left in the caches
    int dir = 0;
    auto turn = [&] { return dir ^= 1; };
    auto turned = [&] {
      SysScal t = SC;
      t.rev = turn();
      return t;
    };
    // y = a x + b D in on the even sites with its reductions red in part
    auto hop_red = [&](Field<R> y, Field<R> in, Field<R> x, Ar a, Ar b, int g5o, double* part, int red, int v,
                       hipStream_t q) -> Parts {
      const int nv = red == 3 ? 3 : 1;
      hop<R>(c, y, in, x, 0, nrhs, lb, colour, a, b, 0, g5o, q,
             nslot ? Fused{part, nlb, nslot, red, live(v), 0, turn()} : Fused{nullptr, 0, 0, 0, live(v), 0, turn()});
      Parts r = {part, nslot};
      if (!nslot) {
        if (red == 3) blas_cdot3<R>(G, nrhs, y, x, y, part, q);
        else blas_norm2<R>(G, nrhs, y, 1, part, q);
        r.n = n1;
      }
      if (r.n > 4096) {      // large lattices with few systems: the consumers would add too many
        r.n = compress_parts(nsys, nv, r, w->partE, q);
        r.p = w->partE;
      }
      return r;
    };
    auto hop_odd = [&](Field<R> in, int g5i, int v, hipStream_t q) {
      hop<R>(c, T, in, NONE, 1, nrhs, lb, colour, Ar(0), Ar(1), g5i, 0, q, Fused{nullptr, 0, 0, 0, live(v), 0, turn()});
    };
    // ITERS_PER_GRAPH iterations on all systems (no host interaction; the state of the systems
    // starts and ends in version 0)
    auto iterate = [&](hipStream_t q) {
      int v = 0;
      Parts last = {nullptr, 0};
      for (int k = 0; k < ITERS_PER_GRAPH; ++k) {
        if (method == SAP_CG) {
          // q = M_hat p ; s -= alpha q (x += alpha p waits for the direction update)
          hop_odd(P, 0, v, q);
          const Parts qq = hop_red(Q, T, P, aI, k2R, 0, w->partA, 1, v, q);
          blas_cg_s<R>(G, nrhs, S, Q, turned(), v, qq, w->partB, q);
          // r = M_hat^dagger s ; x += alpha p, p = r + beta p
          hop_odd(S, 1, v, q);
          const Parts rr = hop_red(Rr, T, S, aI, k2R, 1, w->partC, 1, v, q);
          blas_cg_xp<R>(G, nrhs, Ee, P, Rr, turned(), v, {w->partB, n1}, rr, q);
          v ^= 1;
        } else if (method == SAP_BICGSTAB) {
          // residual r in S, shadow r0 in Rr, v in Q, t in HX
          blas_bicg_p<R>(G, nrhs, P, S, Q, turned(), v, last, q);
          if (last.p) v ^= 1;
          hop_odd(P, 0, v, q);
          hop<R>(c, Q, T, P, 0, nrhs, lb, colour, aI, k2R, 0, 0, q, Fused{nullptr, 0, 0, 0, live(v), 0, turn()});
          blas_cdot3<R>(G, nrhs, Rr, Q, NONE, w->partB, q);
          blas_bicg_s<R>(G, nrhs, S, Q, turned(), v, {w->partB, n1}, w->partD, q);
          v ^= 1;
          hop_odd(S, 0, v, q);
          const Parts ts = hop_red(HX, T, S, aI, k2R, 0, w->partC, 3, v, q);
          blas_bicg_xr<R>(G, nrhs, Ee, P, S, HX, Rr, turned(), v, ts, {w->partD, n1}, w->partA, q);
          v ^= 1;
          last = {w->partA, n1};
        } else {
          // a term: S -> HX -> S (x_e += t on active systems; t <- k^2 D_eo D_oe t)
          const Field<R> from = k & 1 ? HX : S, to = k & 1 ? S : HX;
          blas_geom_add<R>(G, nrhs, Ee, from, turned(), v, last, q);
          if (last.p) v ^= 1;
          hop_odd(from, 0, v, q);
          last = hop_red(to, T, NONE, Ar(0), (Ar)(kap * kap * shift_inv), 0, w->partA, 1, v, q);
        }
      }
      if (method == SAP_CG) fin_count(SC, v, q);
      else if (method == SAP_BICGSTAB) fin_bicg_rho(SC, v, last, 0, q);
      else fin_geom(SC, v, last, 0, q);
    };
    hipGraphExec_t exec = nullptr;
    for (auto& g : w->graphs)
      if (g.nrhs == nrhs && g.lb == lb && g.sel == colour && g.prec == prec_of<R>() && g.method == method &&
          g.rho == rho)
        exec = g.exec;
    if (!exec) {
      hipGraph_t graph;
      if (hipStreamBeginCapture(w->cap, hipStreamCaptureModeThreadLocal) == hipSuccess) {
        iterate(w->cap);
        if (hipStreamEndCapture(w->cap, &graph) == hipSuccess) {
          if (hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0) != hipSuccess) exec = nullptr;
          (void)hipGraphDestroy(graph);
        }
      }
      (void)hipGetLastError();
      if (exec) w->graphs.push_back({nrhs, lb, colour, prec_of<R>(), method, rho, exec});
    }
    for (;;) {
      SAP_HIP_CHECK(c, hipMemcpyAsync(w->h_flags, w->flags, 12, hipMemcpyDeviceToHost, st));
      SAP_HIP_CHECK(c, hipStreamSynchronize(st));
      if (w->h_flags[0])
        return sap_fail(c, SAP_E_NONFINITE,
                        "non-finite value in the inner solve (stage " + std::to_string(w->h_flags[0]) + ")");
      if (w->h_flags[2]) return sap_fail(c, SAP_E_NOCONV, "the geometric series diverges (spectral radius >= 1)");
      if (w->h_flags[1] == 0) break;
      if (total_iters >= o->max_iter) break;
      if (exec) {
        SAP_HIP_CHECK(c, hipGraphLaunch(exec, st));
      } else {
        iterate(st);
      }
      total_iters += ITERS_PER_GRAPH;
    }
    // x_e += e and, in FP64, x_o = b_o + k D_oe x_e, which leaves a residual on the even sites
    // only: r_e = b_e - x_e + k D_eo x_o (even-site systems: r_e = b_e - (1 + rho) x_e +
    // k^2 D_eo D_oe x_e), its norm summed by the hop where its mapping can. The
    // loop is bound by memory, at 24^3x48 with 12 rhs by 1.5 GB fields: correcting both
    // parities, M x and b - M x read and wrote about twice as many. FP16 BiCGstab on 24^3x2
    // blocks (five corrections) 88.8 -> 81.7 ms, FP32 CG (three) 409 -> 404 ms.
    blas_add_resid<R>(G, nrhs, X, Ee, B, R64, 1.0 + rho, st);
    const Field<double> NONE64 = {nullptr, 0, 0};
    if (eo_only) hop<double>(c, AX, X, NONE64, 1, nrhs, lb, colour, 0.0, 1.0, 0, 0, st);
    else hop<double>(c, X, X, B, 1, nrhs, lb, colour, 1.0, kap, 0, 0, st);
    const Field<double> XO = eo_only ? AX : X;
    const double kr = eo_only ? kap * kap : kap;
    int nr = hop_red_slots(hop_args<double>(c, R64, XO, R64, 0, nrhs, lb, colour, 1.0, kr, 0, 0), nlb);
    if ((size_t)nr * nsys > w->part_cap) nr = 0;
    hop<double>(c, R64, XO, R64, 0, nrhs, lb, colour, 1.0, kr, 0, 0, st,
                nr ? Fused{w->partA, nlb, nr, 1} : Fused{});
    if (!nr) {
      blas_norm2<double>(G, nrhs, R64, 1, w->partA, st);
      nr = n1;
    }
    fin_sum(nsys, {w->partA, nr}, w->rnorm2, st);
    SAP_HIP_CHECK(c, hipGetLastError());
  }
  if (info) {
    SAP_HIP_CHECK(c, hipMemcpyAsync(w->h_iters, w->iters, nsys * 4, hipMemcpyDeviceToHost, st));
    SAP_HIP_CHECK(c, hipStreamSynchronize(st));
    for (int s = 0; s < nsys; ++s) {
      const double bb = w->h_bnorm2[s];
      info[s].iters = w->h_selected[s] ? w->h_iters[s] : 0;
      info[s].outer = w->h_selected[s] ? outer : 0;
      info[s].true_rel_res = (w->h_selected[s] && bb > 0) ? std::sqrt(w->h_rnorm2[s] / bb) : 0.0;
    }
  }
  return status;
}

// ---- hop-mapping autotuner -------------------------------------------------------------
template <class R>
static int tune_one(sap_ctx* c, bool full, int nrhs, hipStream_t st, float* us_out) {
  SolverWS* w = ws_of(c);
  typedef typename arith<R>::type Ar;
  const long long Vhp = c->Vhp;
  const bool f16 = std::is_same<R, h16>::value;
  HopArgs<R> A;
  A.out = full_field<R>(w->ax, Vhp);
  A.in = full_field<R>(w->r64, Vhp);
  A.x = full ? A.in : Field<R>{nullptr, 0, 0, 0};
  A.U = gauge_of<R>(c);
  A.g = c->g;
  A.nrhs = nrhs;
  A.parity_out = full ? -1 : 0;
  A.lb = A.slb = 0;
  A.colour = 0;
  A.block = -1;
  A.a = Ar(1);
  A.b = Ar(-c->geom.kappa);
  A.g5_in = A.g5_out = 0;
  hipEvent_t e0, e1;
  SAP_HIP_CHECK(c, hipEventCreate(&e0));
  SAP_HIP_CHECK(c, hipEventCreate(&e1));
  int best = HOP_MAP_SITE, solve = HOP_MAP_SITE;
  float best_ms = 1e30f, solve_ms = 1e30f;
  for (int m = 0; m < HOP_NMAP; ++m) {
    const bool one_rhs_alias = m == HOP_MAP_LANE4 || m == HOP_MAP_WAVE4 ||
                               (m >= HOP_SWEEP && m != HOP_MAP_MARCH1 && m != HOP_MAP_WALK1 &&
                                m != HOP_MAP_BAND1 && m != HOP_MAP_SLAB1 && m != HOP_MAP_SLAB1W &&
                                m != HOP_MAP_SLABD);
    // the LDS-staged slab kernel exists for FP32 and FP16 storage (FP64 runs SLAB1)
    const bool f64_alias = m == HOP_MAP_SLABD && std::is_same<R, double>::value;
    const bool half_only = m == HOP_MAP_STREAM || m >= HOP_MAP_WALK1;
    // FP16 storage has the site and marching kernels only
    const bool f16_alias = f16 && m != HOP_MAP_SITE && m != HOP_MAP_MARCH1 && m != HOP_MAP_MARCH2 && m != HOP_MAP_SLABD &&
                           m != HOP_MAP_MARCH4;
    if ((full && half_only) || (nrhs == 1 && one_rhs_alias) || f16_alias || f64_alias) {
      // the streaming, walking and band kernels exist for half hops only (the full
      // operator runs the walking and band maps as MARCH1 / MARCH2); with one rhs the
      // grouped and sweep orders coincide with SITE, MARCH2 / MARCH4 with MARCH1 and
      // WALK2 with WALK1
      if (us_out) us_out[m] = -1.0f;
      continue;
    }
    // MARCH1 has two kernels in FP32 and FP64, and both are candidates; us_out has the time of the
    // one that its rule picks, as a context would run it with the mapping set by hand. Solves
    // leave the choice to the rule: the register-blocked one adds no reductions, so that they lose more than
    // the hop gains (12x24^3 FP64 1 rhs: hop 18.2 / 18.6 us, series solve of the blocks 2.56 / 2.41 ms).
    const bool two = m == HOP_MAP_MARCH1 && !f16;
    A.map = m;
    int rule = m;
    if constexpr (!std::is_same<R, h16>::value)
      if (two) rule = hop_is_split(A) ? HOP_MAP_MARCH1_SPLIT : HOP_MAP_MARCH1_REG;
    for (int t = 0; t < (two ? 2 : 1); ++t) {
      A.map = two ? HOP_MAP_MARCH1_REG + t : m;
      for (int k = 0; k < 2; ++k) launch_hop<R>(A, st);
      SAP_HIP_CHECK(c, hipEventRecord(e0, st));
      const int reps = 6;
      for (int k = 0; k < reps; ++k) launch_hop<R>(A, st);
      SAP_HIP_CHECK(c, hipEventRecord(e1, st));
      SAP_HIP_CHECK(c, hipEventSynchronize(e1));
      float ms = 0;
      SAP_HIP_CHECK(c, hipEventElapsedTime(&ms, e0, e1));
      ms /= reps;
      if (hipGetLastError() != hipSuccess) ms = 1e30f;   // variant not launchable here
      if (ms < best_ms) { best_ms = ms; best = A.map; }
      if (A.map != rule) continue;
      if (us_out) us_out[m] = ms * 1e3f;
      if (ms < solve_ms) { solve_ms = ms; solve = m; }
    }
  }
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  c->hop_map[full ? 1 : 0][prec_of<R>()][nrhs] = (signed char)best;
  c->hop_tuned[full ? 1 : 0][prec_of<R>()][nrhs] = true;
  if (!full) c->hop_solve[prec_of<R>()][nrhs] = (signed char)solve;
  return SAP_OK;
}

extern "C" int sap_tune(sap_ctx* c, int nrhs, float* us_out, void* stream) {
  if (c && c->solver) drop_graphs(ws_of(c));   // captured graphs hold the old mappings
  if (!c) return sap_fail(nullptr, SAP_E_ARG, "ctx is NULL");
  if (nrhs < 1 || nrhs > c->geom.max_rhs) return sap_fail(c, SAP_E_ARG, "nrhs must be in [1, max_rhs]");
  if (!c->have_gauge) return sap_fail(c, SAP_E_STATE, "no gauge field set");
  hipStream_t st = (hipStream_t)stream;
  SolverWS* w = ws_of(c);
  const size_t fb = (size_t)24 * c->Vhp * nrhs * sizeof(double2);
  SAP_HIP_CHECK(c, hipMemsetAsync(w->r64, 0, fb, st));
  SAP_HIP_CHECK(c, hipMemsetAsync(w->ax, 0, fb, st));
  int rc;
  if ((rc = tune_one<double>(c, true, nrhs, st, us_out ? us_out + 0 * HOP_NMAP : nullptr))) return rc;
  if ((rc = tune_one<float>(c, true, nrhs, st, us_out ? us_out + 1 * HOP_NMAP : nullptr))) return rc;
  if ((rc = tune_one<double>(c, false, nrhs, st, us_out ? us_out + 2 * HOP_NMAP : nullptr))) return rc;
  if ((rc = tune_one<float>(c, false, nrhs, st, us_out ? us_out + 3 * HOP_NMAP : nullptr))) return rc;
  if ((rc = tune_one<h16>(c, true, nrhs, st, us_out ? us_out + 4 * HOP_NMAP : nullptr))) return rc;
  if ((rc = tune_one<h16>(c, false, nrhs, st, us_out ? us_out + 5 * HOP_NMAP : nullptr))) return rc;
  return SAP_OK;
}

extern "C" int sap_set_hop_map(sap_ctx* c, int full, sap_prec prec, int nrhs, int map) {
  if (!c) return sap_fail(nullptr, SAP_E_ARG, "ctx is NULL");
  if (nrhs < 1 || nrhs > 64) return sap_fail(c, SAP_E_ARG, "nrhs must be in [1, 64]");
  if (map < -1 || map >= HOP_NMAP) return sap_fail(c, SAP_E_ARG, "unknown mapping");
  if (full && map == HOP_MAP_STREAM) return sap_fail(c, SAP_E_ARG, "the streaming mapping is for the even-odd hop only");
  if (prec != SAP_F64 && prec != SAP_F32 && prec != SAP_F16) return sap_fail(c, SAP_E_ARG, "unknown precision");
  if (c->solver) drop_graphs(ws_of(c));
  c->hop_map[full ? 1 : 0][prec][nrhs] = (signed char)map;
  c->hop_tuned[full ? 1 : 0][prec][nrhs] = false;
  if (!full) c->hop_solve[prec][nrhs] = (signed char)map;
  return SAP_OK;
}

int sap::check_solve_opts(sap_ctx* c, const sap_solve_opts* o) {
  if (!o) return sap_fail(c, SAP_E_ARG, "opts is NULL");
  if (!(o->tol > 0 && o->tol < 1)) return sap_fail(c, SAP_E_ARG, "tol must be in (0, 1)");
  if (o->max_iter < 1 || o->max_outer < 1) return sap_fail(c, SAP_E_ARG, "max_iter and max_outer must be >= 1");
  if (o->inner_prec != SAP_F64 && o->inner_prec != SAP_F32 && o->inner_prec != SAP_F16)
    return sap_fail(c, SAP_E_ARG, "unknown inner precision");
  if (o->inner_prec != SAP_F64 && !(o->inner_tol > 0 && o->inner_tol < 1))
    return sap_fail(c, SAP_E_ARG, "inner_tol must be in (0, 1) for an FP32 or FP16 inner solve");
  if (o->method != SAP_CG && o->method != SAP_BICGSTAB && o->method != SAP_GEOM && o->method != SAP_SAP_BICGSTAB)
    return sap_fail(c, SAP_E_ARG, "unknown method");
  if (o->sap_block_terms < 0 || o->sap_block_terms > 100000)
    return sap_fail(c, SAP_E_ARG, "sap_block_terms must be in [0, 100000]");
  if (o->method == SAP_SAP_BICGSTAB &&
      (o->sap_ncy < 1 || !(o->sap_block_terms > 0 || (o->inner_tol > 0 && o->inner_tol < 1))))
    return sap_fail(c, SAP_E_ARG,
                    "SAP_SAP_BICGSTAB needs sap_ncy >= 1 and inner_tol in (0, 1) or sap_block_terms > 0");
  return SAP_OK;
}

// ---- Schwarz-preconditioned BiCGstab for M x = b ----------------------------------------
// FP64 BiCGstab on the full lattice, right-preconditioned (M K y = b, x = K y) by K = ncy
// cycles of the multiplicative Schwarz alternating procedure on the level-1 x0 blocks: for
// the black blocks, then the white blocks, y = W1^{-1} (v - M x_K) restricted to that
// colour's blocks (W1 is block diagonal) and x_K += y. The block systems of a colour are one
// batched solve_impl call (CG at inner_prec to the relative residual inner_tol). The few
// outer iterations are driven from the host, which holds the complex scalars.
//
// A full FP64 field [rhs][parity][tiles] is read as 2 * nrhs half fields of stride 12 Vhp,
// so the per-system BLAS kernels apply; the host adds the two parities of every sum.
constexpr int COEF_SLOTS = 8;

struct SapWS {
  int nrhs_cap;
  double2 *r, *r0, *p, *v, *t, *ph, *sh, *kx, *kr, *ky, *mt;
  double2 *g1, *g2;     // series block solves: b_hat (even half), D_oe y (odd half)
  double *part, *dev3, *coef;   // coef, hcoef: COEF_SLOTS sets of coefficients, used in turn
  int slot;
  double *ck_res, *ck_add;   // device coefficients of the preconditioner's two fixed updates
  double *h3, *hcoef;
};

static void sap_ws_free(SapWS* a) {
  void* dev[] = {a->r, a->r0, a->p, a->v, a->t, a->ph, a->sh, a->kx, a->kr, a->ky, a->mt, a->g1, a->g2, a->part, a->dev3,
                 a->coef, a->ck_res, a->ck_add};
  for (void* q : dev)
    if (q) (void)hipFree(q);
  if (a->h3) (void)hipHostFree(a->h3);
  if (a->hcoef) (void)hipHostFree(a->hcoef);
  delete a;
}

extern "C" void sap_sapws_destroy(sap_ctx* c) {
  if (c->sapws) sap_ws_free((SapWS*)c->sapws);
  c->sapws = nullptr;
}

// allocated by sap_create (sap_solver_create); later calls return it
static SapWS* sap_ws(sap_ctx* c) {
  if (c->sapws) return (SapWS*)c->sapws;
  SapWS* a = new SapWS();
  const int n = c->geom.max_rhs;
  a->nrhs_cap = n;
  const size_t fb = (size_t)24 * c->Vhp * n * sizeof(double2);
  const size_t nsys = 2 * (size_t)n;
  const size_t nchunk = (size_t)((c->Vh + TILE - 1) / TILE);
  bool ok = true;
  double2** fields[] = {&a->r, &a->r0, &a->p, &a->v, &a->t, &a->ph, &a->sh, &a->kx, &a->kr, &a->ky, &a->mt,
                        &a->g1, &a->g2};
  for (double2** f : fields) ok = ok && hipMalloc((void**)f, fb) == hipSuccess;
  ok = ok && hipMalloc((void**)&a->part, 3 * nsys * nchunk * 8) == hipSuccess;
  ok = ok && hipMalloc((void**)&a->dev3, 3 * nsys * 8) == hipSuccess;
  ok = ok && hipMalloc((void**)&a->coef, COEF_SLOTS * 6 * nsys * 8) == hipSuccess;
  ok = ok && hipMalloc((void**)&a->ck_res, 6 * nsys * 8) == hipSuccess;
  ok = ok && hipMalloc((void**)&a->ck_add, 6 * nsys * 8) == hipSuccess;
  ok = ok && hipHostMalloc((void**)&a->h3, 3 * nsys * 8, 0) == hipSuccess;
  ok = ok && hipHostMalloc((void**)&a->hcoef, COEF_SLOTS * 6 * nsys * 8, 0) == hipSuccess;
  if (!ok) {
    sap_ws_free(a);
    return nullptr;
  }
  c->sapws = a;
  return a;
}

typedef std::complex<double> zd;

static int sap_bicgstab(sap_ctx* c, double* x, const double* b, int nrhs, const sap_solve_opts* o,
                        sap_solve_info* info, hipStream_t st) {
  SapWS* a = sap_ws(c);
  if (!a) return sap_fail(c, SAP_E_NOMEM, "cannot allocate the Schwarz-preconditioned BiCGstab workspace");
  const long long Vhp = c->Vhp;
  const SysGrid G = make_sysgrid(c->Vh, c->g.V3h, 0, c->geom.L[0], 0, 2 * nrhs);   // full lattice, one block
  const int nh = 2 * nrhs;                                                 // half-field systems
  auto H = [&](double2* f) { return Field<double>{f, 12 * Vhp, 0}; };
  const Field<double> NONE = {nullptr, 0, 0};
  const size_t fullb = (size_t)24 * Vhp * nrhs * sizeof(double2);
  std::vector<zd> rho(nrhs), alpha(nrhs), omega(nrhs);
  std::vector<double> bb(nrhs), rr(nrhs);
  std::vector<int> act(nrhs), its(nrhs, 0);

  // per-rhs sums of the three partials (parities added): s3[r] = (<q, y>, ||y||^2)
  auto sums = [&](std::vector<zd>& dot, std::vector<double>& nrm) -> int {
    fin_sum3(nh, {a->part, G.nchunk}, a->dev3, st);
    SAP_HIP_CHECK(c, hipMemcpyAsync(a->h3, a->dev3, 3 * nh * 8, hipMemcpyDeviceToHost, st));
    SAP_HIP_CHECK(c, hipStreamSynchronize(st));
    for (int r = 0; r < nrhs; ++r) {
      const double* u = a->h3 + 6 * r;
      dot[r] = zd(u[0] + u[3], u[1] + u[4]);
      nrm[r] = u[2] + u[5];
    }
    return SAP_OK;
  };
  // y = c0 y + c1 u + c2 w on every rhs (coefficients per rhs, copied to both parities). An
  // iteration uses four sets of coefficients and waits for its sums after the fourth, so that a
  // set has been consumed long before its slot is written again.
  auto lin3 = [&](double2* y, const double2* u, const double2* w, const double2* q, const std::vector<zd>& c0,
                  const std::vector<zd>& c1, const std::vector<zd>& c2, bool want) -> int {
    const size_t o = (size_t)6 * nh * a->slot;
    a->slot = (a->slot + 1) % COEF_SLOTS;
    for (int r = 0; r < nrhs; ++r)
      for (int par = 0; par < 2; ++par) {
        double* cf = a->hcoef + o + 6 * (2 * r + par);
        cf[0] = c0[r].real(); cf[1] = c0[r].imag();
        cf[2] = c1[r].real(); cf[3] = c1[r].imag();
        cf[4] = c2[r].real(); cf[5] = c2[r].imag();
      }
    SAP_HIP_CHECK(c, hipMemcpyAsync(a->coef + o, a->hcoef + o, 6 * nh * 8, hipMemcpyHostToDevice, st));
    blas_lin3<double>(G, nh, H(y), H((double2*)u), w ? H((double2*)w) : NONE, q ? H((double2*)q) : NONE, a->coef + o,
                      want ? a->part : nullptr, st);
    return SAP_OK;
  };
  auto cdot = [&](const double2* q, const double2* y, const double2* z, std::vector<zd>& dot,
                  std::vector<double>& nrm) -> int {
    blas_cdot3<double>(G, nh, H((double2*)q), H((double2*)y), z ? H((double2*)z) : NONE, a->part, st);
    return sums(dot, nrm);
  };
  const std::vector<zd> one(nrhs, zd(1, 0)), zero(nrhs, zd(0, 0)), mone(nrhs, zd(-1, 0));
  // block solves of the preconditioner
  sap_solve_opts bo = *o;
  bo.tol = o->inner_tol;
  bo.inner_tol = o->inner_prec == SAP_F32   ? std::max(o->inner_tol, 1e-5)
                 : o->inner_prec == SAP_F16 ? std::max(o->inner_tol, 2e-3)
                                            : o->inner_tol;
  bo.max_outer = 40;
  bo.max_iter = 1 << 30;
  bo.method = SAP_CG;
  long long block_iters = 0;
  std::vector<sap_solve_info> binfo((size_t)nrhs * (c->geom.L[0] / c->geom.l0));
  // the preconditioner's fixed updates kr = in - M kx (0, 1, -1) and kx += ky (1, 1, 0),
  // uploaded once so that applying K needs no host synchronisation
  for (int sys = 0; sys < nh; ++sys) {
    const double res_c[6] = {0, 0, 1, 0, -1, 0}, add_c[6] = {1, 0, 1, 0, 0, 0};
    for (int e = 0; e < 6; ++e) {
      a->hcoef[6 * sys + e] = res_c[e];
      a->hcoef[6 * nh + 6 * sys + e] = add_c[e];
    }
  }
  SAP_HIP_CHECK(c, hipMemcpyAsync(a->ck_res, a->hcoef, 6 * nh * 8, hipMemcpyHostToDevice, st));
  SAP_HIP_CHECK(c, hipMemcpyAsync(a->ck_add, a->hcoef + 6 * nh, 6 * nh * 8, hipMemcpyHostToDevice, st));
  SAP_HIP_CHECK(c, hipStreamSynchronize(st));
  const double kap = c->geom.kappa;
  const int lb = c->geom.l0;
  // Y = the first N terms of the even-odd geometric series of W1 y = rhs on the blocks of a
  // colour (Horner form y_e <- b_hat_e + k^2 D_eo D_oe y_e), then y_o = rhs_o + k D_oe y_e; the
  // other blocks of y are set to zero, or (keep, split kernel only) left as they are
  auto series = [&](double2* y, const double2* rhs, int colour, bool keep) {
    const Field<double> RHS = full_field<double>((void*)rhs, Vhp), Y = full_field<double>(y, Vhp);
    const Field<double> BH = full_field<double>(a->g1, Vhp), Z = full_field<double>(a->g2, Vhp);
    const Field<double> NONE64 = {nullptr, 0, 0, 0};
    Fused f;
    f.keep = keep;
    const int N = o->sap_block_terms;
    hop<double>(c, N == 1 ? Y : BH, RHS, RHS, 0, nrhs, lb, colour, 1.0, kap, 0, 0, st, f);
    for (int n = 1; n < N; ++n) {
      hop<double>(c, Z, n == 1 ? BH : Y, NONE64, 1, nrhs, lb, colour, 0.0, 1.0, 0, 0, st, f);
      hop<double>(c, Y, Z, BH, 0, nrhs, lb, colour, 1.0, kap * kap, 0, 0, st, f);
    }
    hop<double>(c, Y, Y, RHS, 1, nrhs, lb, colour, 1.0, kap, 0, 0, st, f);
  };
  // the argument of a hop of the colour's sites only, all hops of M kept
  auto on_colour = [&](double2* out, const double2* in, const double2* x, double b, int colour) {
    HopArgs<double> A = hop_args<double>(c, full_field<double>(out, Vhp), full_field<double>((void*)in, Vhp),
                                         full_field<double>((void*)x, Vhp), -1, nrhs, 0, colour, 1.0, b, 0, 0);
    A.slb = lb;
    A.map = hop_map_for(c, true, SAP_F64, nrhs, hop_use(c->g, lb, A.colour, A.block));
    return A;
  };
  // with series block solves on the split kernel, a cycle's first two block steps write their
  // sites of out in place: out vanishes on the colour being solved, so that its right-hand side
  // is in + k D out on that colour
  const HopArgs<double> probe = hop_args<double>(c, {}, {}, {}, 0, nrhs, lb, SAP_WHITE, 1.0, kap, 0, 0);
  const bool in_place = o->sap_block_terms > 0 && hop_is_split(probe);
  // out = K in
  auto K = [&](double2* out, const double2* in) -> int {
    double2* kx = in_place ? out : a->kx;
    if (!in_place) SAP_HIP_CHECK(c, hipMemsetAsync(kx, 0, fullb, st));
    for (int cyc = 0; cyc < o->sap_ncy; ++cyc)
      for (int col = 0; col < 2; ++col) {
        const int colour = col == 0 ? SAP_BLACK : SAP_WHITE;
        const double2* rhs = in;
        if (in_place && cyc == 0 && col > 0) {
          launch_hop<double>(on_colour(a->kr, kx, in, kap, colour), st);
          rhs = a->kr;
        } else if (cyc > 0 || col > 0) {
          // in - M kx on the colour's sites
          launch_hop<double>(on_colour(a->mt, kx, kx, -kap, colour), st);
          blas_lin3<double>(G, nh, H(a->kr), H((double2*)in), H(a->mt), NONE, a->ck_res, nullptr, st);
          rhs = a->kr;
        }
        if (in_place && cyc == 0) {
          series(kx, rhs, colour, col > 0);
          SAP_HIP_CHECK(c, hipGetLastError());
          continue;
        }
        if (o->sap_block_terms > 0) {
          series(a->ky, rhs, colour, false);
          SAP_HIP_CHECK(c, hipGetLastError());
        } else {
          const double* r64 = (const double*)rhs;
          int rc = o->inner_prec == SAP_F64
                       ? solve_impl<double>(c, (double*)a->ky, r64, nrhs, lb, colour, &bo, binfo.data(), st)
                   : o->inner_prec == SAP_F32
                       ? solve_impl<float>(c, (double*)a->ky, r64, nrhs, lb, colour, &bo, binfo.data(), st)
                       : solve_impl<h16>(c, (double*)a->ky, r64, nrhs, lb, colour, &bo, binfo.data(), st);
          if (rc) return rc;
          for (auto& e : binfo) block_iters += e.iters;
        }
        blas_lin3<double>(G, nh, H(kx), H(a->ky), NONE, NONE, a->ck_add, nullptr, st);
        SAP_HIP_CHECK(c, hipGetLastError());
      }
    if (kx != out) SAP_HIP_CHECK(c, hipMemcpyAsync(out, kx, fullb, hipMemcpyDeviceToDevice, st));
    return SAP_OK;
  };

  SAP_HIP_CHECK(c, hipMemsetAsync(x, 0, fullb, st));
  {
    std::vector<zd> d(nrhs);
    int rc = cdot((const double2*)b, (const double2*)b, nullptr, d, bb);
    if (rc) return rc;
    for (int r = 0; r < nrhs; ++r) bb[r] = d[r].real();
  }
  const double tol2 = o->tol * o->tol;
  int status = SAP_OK, restarts = 0;
  long long total = 0;
  for (;;) {
    // r = b - M x ; r0 = r
    int rc = apply_op_any(c, a->mt, x, nrhs, 0, 0, -1, SAP_F64, st);
    if (rc) return rc;
    SAP_HIP_CHECK(c, hipMemcpyAsync(a->r, b, fullb, hipMemcpyDeviceToDevice, st));
    std::vector<zd> rn(nrhs);
    if ((rc = lin3(a->r, a->mt, nullptr, a->r, one, mone, zero, true))) return rc;
    if ((rc = sums(rn, rr))) return rc;
    bool done = true, finite = true;
    for (int r = 0; r < nrhs; ++r) {
      if (!std::isfinite(rr[r])) finite = false;
      act[r] = bb[r] > 0 && rr[r] > tol2 * bb[r];
      if (act[r]) done = false;
    }
    if (!finite) { status = sap_fail(c, SAP_E_NONFINITE, "non-finite residual"); break; }
    if (done) break;
    if (restarts >= o->max_outer || total >= o->max_iter) {
      status = sap_fail(c, SAP_E_NOCONV, "solver did not reach tol within max_outer / max_iter");
      break;
    }
    ++restarts;
    SAP_HIP_CHECK(c, hipMemcpyAsync(a->r0, a->r, fullb, hipMemcpyDeviceToDevice, st));
    SAP_HIP_CHECK(c, hipMemsetAsync(a->p, 0, fullb, st));
    SAP_HIP_CHECK(c, hipMemsetAsync(a->v, 0, fullb, st));
    for (int r = 0; r < nrhs; ++r) rho[r] = alpha[r] = omega[r] = zd(1, 0);
    // rn holds <r0, r> = ||r||^2 at the start
    for (int r = 0; r < nrhs; ++r) rn[r] = zd(rr[r], 0);
    while (total < o->max_iter) {
      bool any = false;
      std::vector<zd> beta(nrhs), mbo(nrhs);
      for (int r = 0; r < nrhs; ++r) {
        if (act[r] && (rr[r] <= tol2 * bb[r] || std::abs(rho[r]) == 0 || std::abs(omega[r]) == 0 ||
                       std::abs(rn[r]) == 0))
          act[r] = 0;
        beta[r] = act[r] ? (rn[r] / rho[r]) * (alpha[r] / omega[r]) : zd(0, 0);
        mbo[r] = -beta[r] * omega[r];
        if (act[r]) rho[r] = rn[r];
        any = any || act[r];
      }
      if (!any) break;
      // p = r + beta (p - omega v) ; ph = K p ; v = M ph
      if ((rc = lin3(a->p, a->r, a->v, nullptr, beta, one, mbo, false))) return rc;
      if ((rc = K(a->ph, a->p))) return rc;
      if ((rc = apply_op_any(c, a->v, a->ph, nrhs, 0, 0, -1, SAP_F64, st))) return rc;
      std::vector<zd> den(nrhs), ma(nrhs), dts(nrhs), mo(nrhs), al_c(nrhs), om_c(nrhs);
      std::vector<double> dummy(nrhs), tt(nrhs);
      if ((rc = cdot(a->r0, a->v, nullptr, den, dummy))) return rc;
      for (int r = 0; r < nrhs; ++r) {
        if (act[r] && std::abs(den[r]) == 0) act[r] = 0;
        alpha[r] = act[r] ? rho[r] / den[r] : zd(0, 0);
        ma[r] = -alpha[r];
      }
      // s = r - alpha v (in r) ; sh = K s ; t = M sh ; omega = <t, s> / <t, t>
      if ((rc = lin3(a->r, a->v, nullptr, nullptr, one, ma, zero, false))) return rc;
      if ((rc = K(a->sh, a->r))) return rc;
      if ((rc = apply_op_any(c, a->t, a->sh, nrhs, 0, 0, -1, SAP_F64, st))) return rc;
      if ((rc = cdot(a->t, a->r, a->t, dts, tt))) return rc;
      for (int r = 0; r < nrhs; ++r) {
        omega[r] = (act[r] && tt[r] > 0) ? dts[r] / tt[r] : zd(0, 0);
        mo[r] = -omega[r];
        al_c[r] = alpha[r];
        om_c[r] = omega[r];
        if (act[r]) its[r] += 1;
      }
      // x += alpha ph + omega sh ; r = s - omega t, with <r0, r> and ||r||^2
      if ((rc = lin3((double2*)x, a->ph, a->sh, nullptr, one, al_c, om_c, false))) return rc;
      if ((rc = lin3(a->r, a->t, nullptr, a->r0, one, mo, zero, true))) return rc;
      if ((rc = sums(rn, rr))) return rc;
      for (int r = 0; r < nrhs; ++r)
        if (!std::isfinite(rr[r])) return sap_fail(c, SAP_E_NONFINITE, "non-finite value in BiCGstab");
      ++total;
    }
  }
  if (info) {
    // true residuals (the loop above ends with them in rr)
    for (int r = 0; r < nrhs; ++r) {
      info[r].iters = its[r];
      info[r].outer = restarts;
      info[r].true_rel_res = bb[r] > 0 ? std::sqrt(rr[r] / bb[r]) : 0.0;
    }
  }
  (void)block_iters;
  return status;
}

// (M_hat + rho) x_e = b_e on the blocks of length lb (0: full lattice), even sites only
int sap_solve_eo_shift(sap_ctx* c, double* x, const double* b, int nrhs, int lb, double rho,
                       const sap_solve_opts* o, sap_solve_info* info, hipStream_t st) {
  if (o->method == SAP_SAP_BICGSTAB) return sap_fail(c, SAP_E_ARG, "SAP_SAP_BICGSTAB solves M x = b only");
  if (o->inner_prec == SAP_F64) return solve_impl<double>(c, x, b, nrhs, lb, 0, o, info, st, rho, true);
  if (o->inner_prec == SAP_F32) return solve_impl<float>(c, x, b, nrhs, lb, 0, o, info, st, rho, true);
  return solve_impl<h16>(c, x, b, nrhs, lb, 0, o, info, st, rho, true);
}

int sap_solve_any(sap_ctx* c, double* x, const double* b, int nrhs, int lb, int colour,
                  const sap_solve_opts* o, sap_solve_info* info, hipStream_t st) {
  if (o->method == SAP_SAP_BICGSTAB) {
    if (lb != 0) return sap_fail(c, SAP_E_ARG, "SAP_SAP_BICGSTAB solves the full lattice only");
    return sap_bicgstab(c, x, b, nrhs, o, info, st);
  }
  if (o->inner_prec == SAP_F64) return solve_impl<double>(c, x, b, nrhs, lb, colour, o, info, st);
  if (o->inner_prec == SAP_F32) return solve_impl<float>(c, x, b, nrhs, lb, colour, o, info, st);
  return solve_impl<h16>(c, x, b, nrhs, lb, colour, o, info, st);
}

extern "C" {

int solve_full(sap_ctx* c, double* x, const double* b, int nrhs, const sap_solve_opts* o,
               sap_solve_info* info, void* stream) {
  if (!c) return sap_fail(nullptr, SAP_E_ARG, "ctx is NULL");
  if (!x || !b) return sap_fail(c, SAP_E_ARG, "x or b is NULL");
  if (x == b) return sap_fail(c, SAP_E_ARG, "x and b must not alias");
  if (nrhs < 1 || nrhs > c->geom.max_rhs) return sap_fail(c, SAP_E_ARG, "nrhs must be in [1, max_rhs]");
  int rc = check_solve_opts(c, o);
  if (rc) return rc;
  if (!c->have_gauge) return sap_fail(c, SAP_E_STATE, "no gauge field set");
  return sap_solve_any(c, x, b, nrhs, 0, 0, o, info, (hipStream_t)stream);
}

int solve_blocks(sap_ctx* c, double* x, const double* b, int nrhs, int level, sap_color color, int block,
                 const sap_solve_opts* o, sap_solve_info* info, void* stream) {
  if (!c) return sap_fail(nullptr, SAP_E_ARG, "ctx is NULL");
  if (!x || !b) return sap_fail(c, SAP_E_ARG, "x or b is NULL");
  if (x == b) return sap_fail(c, SAP_E_ARG, "x and b must not alias");
  if (nrhs < 1 || nrhs > c->geom.max_rhs) return sap_fail(c, SAP_E_ARG, "nrhs must be in [1, max_rhs]");
  int lb;
  if (level == 1) lb = c->geom.l0;
  else if (level == 2 && c->geom.l0_sub > 0) lb = c->geom.l0_sub;
  else return sap_fail(c, SAP_E_ARG, "level must be 1, or 2 with l0_sub set");
  if (color != SAP_ALL && color != SAP_BLACK && color != SAP_WHITE)
    return sap_fail(c, SAP_E_ARG, "unknown colour");
  if (block < -1 || block >= c->geom.L[0] / lb) return sap_fail(c, SAP_E_ARG, "block out of range");
  int rc = check_solve_opts(c, o);
  if (rc) return rc;
  if (!c->have_gauge) return sap_fail(c, SAP_E_STATE, "no gauge field set");
  const int sel = block >= 0 ? 3 + block : (int)color;
  return sap_solve_any(c, x, b, nrhs, lb, sel, o, info, (hipStream_t)stream);
}

}  // extern "C"
