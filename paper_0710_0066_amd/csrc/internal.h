// Host-side internals of libsapmi: the context, field descriptors and the launchers
// each translation unit provides.
#pragma once
#include <hip/hip_runtime.h>
#include <string>
#include <type_traits>
#include <vector>
#include "../../include/sapmi.h"
#include "device_common.h"

namespace sap {

// A spinor field in the library layout: element (rhs, parity, component c, site j) of
// complex type at  ptr + rhs*rs + parity*ps + sidx<R>(j, c)  (in complex numbers;
// tiled(j, c, 12) for FP64 and FP16, pairs of components per 16-byte word for FP32).
// Full fields: rs = 24*Vhp, ps = 12*Vhp. Single-parity fields: rs = 12*Vhp, ps = 0.
// FP16 (h16) fields also hold one FP32 norm per site: the components are stored divided
// by it, and the norms of (rhs, parity) start at  (float*)(ptr + rhs*rs + no) + parity*Vhp.
// Full FP16 fields: rs = 26*Vhp, ps = 12*Vhp, no = 24*Vhp; single-parity: rs = 13*Vhp,
// ps = 0, no = 12*Vhp (a half2 and a float are both 4 bytes).
// Gauge field: link (parity p, site j, mu, entry e = 3*row + col) at
//   p*36*Vhp + tiled(j, 9*mu + e, 36)   (FP64);
// the copies the FP32 and FP16 hop kernels read hold rows 0 and 1 only (e < 6), at
// p*24*Vhp + tiled(j, 6*mu + e, 24) (FP32: the entries of a tile row stored in pairs, one
// 16-byte word per lane; FP16: a quad and a pair of entries per link, see
// gauge_to_f32_kernel), and the kernels rebuild row 2 from
// unitarity and unit determinant.
// Momenta / forces (float64): (p, j, mu, a) at  p*32*Vhp + tiled(j, 8*mu + a, 32).
template <class R> struct Field {
  typename vec2<R>::type* ptr;
  long long rs;
  long long ps;
  long long no;            // FP16 only: offset of the norms in an rhs block (complex units)
};

// field descriptors of the library's full and single-parity fields for storage type S
template <class S> inline Field<S> full_field(void* p, long long Vhp) {
  if constexpr (std::is_same<S, h16>::value) return {(typename vec2<S>::type*)p, 26 * Vhp, 12 * Vhp, 24 * Vhp};
  else return {(typename vec2<S>::type*)p, 24 * Vhp, 12 * Vhp, 0};
}
template <class S> inline Field<S> half_field(void* p, long long Vhp) {
  if constexpr (std::is_same<S, h16>::value) return {(typename vec2<S>::type*)p, 13 * Vhp, 0, 12 * Vhp};
  else return {(typename vec2<S>::type*)p, 12 * Vhp, 0, 0};
}
// bytes of nrhs full / single-parity fields
template <class S> inline size_t full_bytes(long long Vhp, int nrhs) {
  if constexpr (std::is_same<S, h16>::value) return (size_t)26 * Vhp * nrhs * 4;
  else return (size_t)24 * Vhp * nrhs * sizeof(typename vec2<S>::type);
}
template <class S> inline size_t half_bytes(long long Vhp, int nrhs) {
  if constexpr (std::is_same<S, h16>::value) return (size_t)13 * Vhp * nrhs * 4;
  else return (size_t)12 * Vhp * nrhs * sizeof(typename vec2<S>::type);
}

template <class R> struct HopArgs {
  Field<R> out, in, x;     // out = a*x + b*D(in); x.ptr may be null
  const typename vec2<R>::type* U;   // gauge field in the tiled layout
  Geo g;
  int nrhs;
  int parity_out;          // -1: both parities (full operator); 0/1: that parity only
  int lb;                  // hops between x0 blocks of this length are dropped (0: none)
  int slb;                 // output restricted to x0 blocks of this length (0: all sites)
  int colour;              // selection for slb: 0 all, 1 black (odd b), 2 white (even b)
  int block;               // >= 0: only this block (colour ignored)
  typename arith<R>::type a, b;
  int g5_in, g5_out;       // multiply the hop input / the hop result by gamma_5
  int map;                 // work-item mapping (HOP_MAP_*), nrhs > 1 only
  // optional (half hop, mappings with hop_red_slots > 0): per-system partial reductions of
  // the output over systems (rhs, block of nlb slices), nslot partials per system:
  //   red = 1: ||out||^2 at npart[sys * nslot + k];
  //   red = 3: (Re, Im <out, x>, ||out||^2) with out conjugated, at
  //   npart[3 (sys * nslot + k) + i].
  double* npart = nullptr;
  int nlb = 0, nslot = 0, red = 0;
  // optional: nonzero where a system (rhs, x0 block; the blocks of slb, or the whole lattice) is
  // still iterated; the output of the others may be left as it is (it is by the split, marching,
  // slab and FP16 kernels; the other mappings compute it)
  const int* active = nullptr;
  int keep = 0;            // split kernel: leave unselected sites as they are (else zero)
  int rev = 0;             // split kernel, linear order: walk the lattice backwards
};

// has every system of the rhs r0 .. r0 + nr - 1 in the slices xa .. xb - 1 converged
// (HopArgs::active)? Such workgroups end at once: a graph of eight iterations runs up to seven
// past the last system's end. FP16 BiCGstab on 24^3x48, 12 rhs, 24^3x2 blocks (corrections of
// nine or ten iterations) 106 -> 91 ms, FP32 CG on 16^3x32 with one rhs 7.87 -> 7.67 ms.
template <class R>
__device__ __forceinline__ bool hop_idle(const HopArgs<R>& A, int r0, int nr, int xa, int xb) {
  if (!A.active) return false;
  const int len = A.slb ? A.slb : A.g.L0, nblk = A.g.L0 / len;
  for (int r = r0; r < r0 + nr; ++r)
    for (int b = xa / len; b <= (xb - 1) / len; ++b)
      if (A.active[r * nblk + b]) return false;
  return true;
}

// Work-item mappings of the hop kernel for several right-hand sides.
enum { HOP_MAP_SITE = 0,    // split kernel: a site's eight hops on eight wavefronts (FP16: one
                            // (site, rhs) per work-item on larger launches), rhs-fastest
       HOP_MAP_LANE4 = 1,   // wavefront = 16 sites x 4 rhs: four lanes share each link load
       HOP_MAP_WAVE4 = 2,   // workgroup = 64 sites x 4 rhs, one rhs per wavefront
       HOP_MAP_STREAM = 3,  // half hop only: x0-streaming, input slice staged in LDS
       HOP_SWEEP = 4,       // added to SITE/LANE4/WAVE4: workgroups rhs(-group)-slowest, so
                            // each rhs sweeps the lattice like a single-rhs launch
       HOP_MAP_REG2 = 7,    // one work-item per site for 2 rhs held in registers: each
       HOP_MAP_REG4 = 8,    //   link is loaded once and applied to 2 (4) rhs
       HOP_MAP_REG2_SWEEP = 9,   // REG2 / REG4 with workgroups group-slowest: each group
       HOP_MAP_REG4_SWEEP = 10,  //   of rhs sweeps the lattice like a small-rhs launch
       HOP_MAP_MARCH1 = 11, // x0-marching: each XCD owns 1/8 of every x0 slice and walks the
       HOP_MAP_MARCH2 = 12, //   slices in order, 1 / 2 / 4 rhs per work-item (any nrhs for
       HOP_MAP_MARCH4 = 13, //   MARCH1)
       HOP_MAP_WALK1 = 14,  // even-odd hop only: x0-walking, time neighbours carried in
       HOP_MAP_WALK2 = 15,  //   registers, 1 / 2 rhs per work-item
       HOP_MAP_BAND1 = 16,  // even-odd hop only: each XCD owns a band of x0 slices, time
                            //   hops carried in registers, 1 rhs per work-item
       HOP_MAP_SLAB1 = 17,  // even-odd hop only: band order, a workgroup owns a spatial tile
       HOP_MAP_SLAB1W = 18, //   of the slice staged in LDS and walks the band; 1 rhs per
       HOP_MAP_SLAB2 = 19,  //   work-item (SLAB1W: tiles up to twice as large), or 2 (SLAB2)
       HOP_MAP_SLABD = 20,  // even-odd FP32 / FP16 hop only: the slab order with the slice
                            //   and its x1 / x2 halo staged in LDS by direct memory-to-LDS
                            //   loads, 1 rhs per work-item (FP64: as SLAB1)
       HOP_NMAP = 21,
       // MARCH1 (FP32 / FP64) with its kernel fixed, as the autotuner may choose: the register-
       // blocked or the split one
       HOP_MAP_MARCH1_REG = 21, HOP_MAP_MARCH1_SPLIT = 22 };
constexpr int HOP_WALK_T = 8;   // slices per walk

template <class R> void launch_hop(const HopArgs<R>& A, hipStream_t s);
// mapping of an untuned context for the full operator or the half hop (prec: sap_prec)
int hop_default_map(const Geo& g, bool full, int prec, int nrhs, int use);
// what a launch computes: all sites, the blocks of a colour (as many in every eighth of x0, or
// not), one block; or a half hop of a solve, which leaves out converged systems
enum { HOP_ALL, HOP_EVENLY, HOP_UNEVENLY, HOP_BLOCK, HOP_SOLVE };
inline int hop_use(const Geo& g, int slb, int colour, int block) {
  if (slb && block >= 0) return HOP_BLOCK;
  if (!slb || colour == 0) return HOP_ALL;
  return g.L0 % (16 * slb) == 0 ? HOP_EVENLY : HOP_UNEVENLY;
}
// does the launch A run the split kernel?
template <class R> bool hop_is_split(const HopArgs<R>& A);
// do the workgroups of the half hop A give each XCD a range of the whole lattice (linear order,
// every block)?
template <class R> bool hop_in_ranges(const HopArgs<R>& A);
template <> bool hop_in_ranges<h16>(const HopArgs<h16>& A);   // half.hip
// partials per system of nlb slices that the half hop A (its mapping, precision, lattice and
// rhs) can write of its output (HopArgs::npart); 0: its mapping has none
template <class R> int hop_red_slots(const HopArgs<R>& A, int nlb);
template <> int hop_red_slots<h16>(const HopArgs<h16>& A, int nlb);   // half.hip
// those of the LDS-staged slab kernel
int slabd_norm_slots(const Geo& g, int nlb);
// the LDS-staged slab kernel on FP16 storage (even-odd hop; dslash.hip)
void launch_slabd16(const HopArgs<h16>& A, hipStream_t s);
template <> void launch_hop<h16>(const HopArgs<h16>& A, hipStream_t s);   // half.hip

// layout conversions
template <class R>
void launch_pack_spinor(const Geo& g, typename vec2<R>::type* out, const double2* in, int nrhs,
                        hipStream_t s);
template <class R>
void launch_unpack_spinor(const Geo& g, double2* out, const typename vec2<R>::type* in,
                          int nrhs, hipStream_t s);
// canonical links -> the context's FP64 links and their reduced copies, with one partial per
// workgroup (load_gauge_parts(g)) of the largest deviation from SU(3)
int load_gauge_parts(const Geo& g);
void launch_load_gauge(const Geo& g, double2* U64, float2* U32, __half2* U16, const double2* in, double* part,
                       hipStream_t s);
void launch_unpack_gauge(const Geo& g, double2* out, const double2* U64, hipStream_t s);
// the reduced link copies of the hop kernels from the FP64 links: two-row FP32 and FP16
// copies, then the three-row FP16 copy of the LDS-staged FP16 hop (layouts in layout.hip)
void launch_gauge_to_f32(const Geo& g, float2* U32, __half2* U16, const double2* U64, hipStream_t s);
void launch_pack_spinor16(const Geo& g, __half2* out, const double2* in, int nrhs, hipStream_t s);
void launch_unpack_spinor16(const Geo& g, double2* out, const __half2* in, int nrhs, hipStream_t s);
void launch_pack_momenta(const Geo& g, double* out, const double* in, hipStream_t s);
void launch_unpack_momenta(const Geo& g, double* out, const double* in, hipStream_t s);

inline Geo make_geo(const int L[4]) {
  Geo g;
  g.L0 = L[0]; g.L1 = L[1]; g.L2 = L[2]; g.L3 = L[3];
  g.L3h = L[3] / 2;
  g.V3h = L[1] * L[2] * L[3] / 2;
  g.Vh = (long long)L[0] * L[1] * L[2] * L[3] / 2;
  g.Vhp = (g.Vh + TILE - 1) / TILE * TILE;
  return g;
}

}  // namespace sap

struct sap_ctx {
  sap_geom geom;
  sap::Geo g;
  long long V, Vh, Vhp;
  int device;
  bool have_gauge;
  double su3_dev;   // largest deviation from SU(3) of the links that were loaded
  double2* U64;   // tiled gauge layout, 72*Vhp complex (whole links: forces, link updates; the FP64
                  // hop kernels read the first two rows of each)
  float2* U32;    // two-row FP32 copy
  __half2* U16;   // two-row FP16 copy (48*Vhp), then the three-row FP16 copy (72*Vhp) the
                  // LDS-staged FP16 hop reads (all copies kept in step with U64)
  std::string err;
  void* solver;   // solver workspace (solver.hip)
  void* forces;   // force / trajectory workspace (hmc.hip)
  void* sapws;    // Schwarz-preconditioned BiCGstab workspace (solver.hip), allocated by sap_create
  // tuned or set hop mapping per [full operator?][precision (sap_prec)][nrhs] (-1: neither),
  // whether it was tuned, and that of the half hops of a solve
  signed char hop_map[2][3][65];
  bool hop_tuned[2][3][65];
  signed char hop_solve[3][65];
};

// largest deviation from SU(3) (|U U^+ - 1| entries, |det U - 1|) sap_set_gauge accepts
constexpr double SAP_SU3_TOL = 1e-10;
// links nearer than this to SU(3) are rounded FP64 matrices: their largest deviation is 1.3e-15
// after a reunitarisation, 5e-15 for exponentials from eigenvectors (16^3x32)
constexpr double SAP_SU3_ROUNDED = 1e-14;

// precision code (sap_prec) of a storage type
template <class S> constexpr int prec_of() {
  return std::is_same<S, double>::value ? SAP_F64 : std::is_same<S, float>::value ? SAP_F32 : SAP_F16;
}

// mapping used for a hop launch: the tuned (or set) one, else the rule on the lattice, the
// precision and the number of rhs. The tuner times launches on every site; the full operator on
// some of the blocks goes by the rule (24^3x48 in FP32, one block, one rhs: 22.6 us with the
// mapping tuned for the whole lattice, 13.8 by the rule).
inline int hop_map_for(const sap_ctx* c, bool full, int prec, int nrhs, int use) {
  const int n = nrhs > 64 ? 64 : nrhs, m = use == sap::HOP_SOLVE ? c->hop_solve[prec][n] : c->hop_map[full][prec][n];
  const bool part = full && (use == sap::HOP_EVENLY || use == sap::HOP_UNEVENLY || use == sap::HOP_BLOCK);
  if (m >= 0 && !(part && c->hop_tuned[full][prec][n])) return m;
  return sap::hop_default_map(c->g, full, prec, nrhs, use);
}

// error helpers (api.hip)
int sap_fail(sap_ctx* ctx, int code, const std::string& msg);
#define SAP_HIP_CHECK(ctx, call)                                                     \
  do {                                                                               \
    hipError_t e_ = (call);                                                          \
    if (e_ != hipSuccess)                                                            \
      return sap_fail((ctx), SAP_E_HIP, std::string(#call) + ": " + hipGetErrorString(e_)); \
  } while (0)

namespace sap {
// validation of solve options shared by every entry point that solves (solver.hip)
int check_solve_opts(sap_ctx* c, const sap_solve_opts* o);
}

// the context's link copy for storage type S
template <class S> inline const typename sap::vec2<S>::type* gauge_of(const sap_ctx* c) {
  if constexpr (std::is_same<S, double>::value) return c->U64;
  else if constexpr (std::is_same<S, float>::value) return c->U32;
  else return c->U16;
}
