// Solver kernels for gfx950.  One tick = k_row -> k_col over all listed slots
// of a handle; the row kernel first advances each slot's control block by the
// controller step of the previous tick, and a block of ticks ends with
// k_close (the controller step of its last tick).
// Every kernel looks up the phase of its slot and does that phase's share of
// the work (or returns).
//
// Data layout (per slot, real = float or double):
//   real planes [ny][nx]; tensors as 3 planes (xx, yy, xy)
//   spectrum: complex [C][nx/2][ny] -- the half spectrum of each plane,
//             stored transposed (one contiguous run of ny per kx) so the
//             column kernel reads and writes whole columns; kx = 0 holds
//             X[0] + i X[nx/2] (both columns of a real row transform are
//             real-valued per row, so they share one complex column).
//
// Row kernels: a work-group owns R consecutive rows of one slot and all C
// components; a column kernel work-group owns W consecutive kx columns.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <mutex>
#include <type_traits>

#include "spff.h"
#include "spff_device.hpp"
#include "spff_engine.hpp"
#include "spff_launch.hpp"

namespace spff {

constexpr int THREADS = 256;
constexpr int MAXE = 8;   // FFT elements per thread per chunk: M <= 2048
constexpr int PAD = 1;    // complex padding per LDS row (bank spread)
constexpr double TWO_PI = 6.283185307179586476925286766559;

// Row-kernel coordinates (row group g, list index si) of this work-group.
// Work-groups are dispatched to the 8 XCDs round-robin by linear id; the
// remap gives consecutive row groups of a slot to one XCD, so the short
// transposed spectrum segments of neighbouring groups (R rows each) meet in
// the same L2 and leave it as whole lines.
__device__ __forceinline__ void row_coords(int ngr, int& g, int& si) {
  const int N = gridDim.x * gridDim.y;
  int L = blockIdx.x + blockIdx.y * gridDim.x;
  if ((N & 7) == 0) L = (L & 7) * (N >> 3) + (L >> 3);
  const int lg = ilog2(ngr);  // ngr is a power of two
  si = L >> lg;
  g = L & (ngr - 1);
}

// Field and spectrum accesses go through global-address-space pointers: the
// slot's field pointers are read from the pointer table, so the compiler
// cannot tell they address device memory and would use flat instructions,
// whose completion it can only wait for all at once (a flat access may be an
// LDS access).  Global loads complete in order and are waited for one by
// one, so the loads of a prologue overlap the arithmetic on the first ones.
#define SPFF_GLOBAL __attribute__((address_space(1)))

template <typename real>
struct V2 {
  real a, b;
};

template <typename real>
struct Pair;
template <>
struct Pair<float> {
  typedef float type __attribute__((ext_vector_type(2)));
};
template <>
struct Pair<double> {
  typedef double type __attribute__((ext_vector_type(2)));
};
// A pixel of a plane: a lane's byte offset plus a displacement in elements
// that is known at compile time.  With the plane's base in scalar registers
// this is the address form base + 32-bit lane offset + immediate: one vector
// register addresses every plane and pixel pair of a lane (64-bit lane
// addresses took more registers than the data and set the row kernels'
// occupancy).  A plane holds less than 4 GiB.
struct At {
  unsigned b;
  int d;
};
__device__ __forceinline__ At operator+(At o, int d) { return {o.b, o.d + d}; }
template <typename real>
__device__ __forceinline__ At at(int o) {
  return {(unsigned)o * (unsigned)sizeof(real), 0};
}
template <typename T>
__device__ __forceinline__ SPFF_GLOBAL T* gat(const void* p, unsigned b, int disp) {
  return (SPFF_GLOBAL T*)((SPFF_GLOBAL char*)const_cast<void*>(p) + b + disp);
}
template <typename real>
__device__ __forceinline__ V2<real> ld2(const real* p, At o) {
  using T = typename Pair<real>::type;
  const T v = *gat<const T>(p, o.b, o.d * (int)sizeof(real));
  return {v.x, v.y};
}
template <typename real>
__device__ __forceinline__ void st2(real* p, At o, real a, real b) {
  using T = typename Pair<real>::type;
  T v;
  v.x = a;
  v.y = b;
  *gat<T>(p, o.b, o.d * (int)sizeof(real)) = v;
}
// one complex value of a spectrum, element i + d (d known at compile time)
template <typename real>
__device__ __forceinline__ cplx<real> ldc(const cplx<real>* p, unsigned i, int d = 0) {
  using T = typename Pair<real>::type;
  const T v = *gat<const T>(p, i * (unsigned)sizeof(T), d * (int)sizeof(T));
  return mk<cplx<real>>(v.x, v.y);
}
template <typename real>
__device__ __forceinline__ void stc(cplx<real>* p, unsigned i, const cplx<real>& c, int d = 0) {
  using T = typename Pair<real>::type;
  T v;
  v.x = c.x;
  v.y = c.y;
  *gat<T>(p, i * (unsigned)sizeof(T), d * (int)sizeof(T)) = v;
}
// active-set bytes of a pixel pair (even pixel first)
template <typename real>
__device__ __forceinline__ unsigned short ldm(const unsigned char* p, At o) {
  return *gat<const unsigned short>(p, o.b / (unsigned)sizeof(real), o.d);
}
template <typename real>
__device__ __forceinline__ void stm(unsigned char* p, At o, bool a, bool b) {
  *gat<unsigned short>(p, o.b / (unsigned)sizeof(real), o.d) = (unsigned short)((a ? 1u : 0u) | (b ? 0x100u : 0u));
}

template <typename real>
__device__ __forceinline__ real lower_bound(real pref, const SlotParam& P) {
  if (P.irr == 1) return pref;
  return pref >= real(P.threshold) ? pref : real(0);
}

// What a row kernel does in one pass over its rows: finish the previous
// tick's phase (its pointwise part works on inverse-transformed rows) and
// start the next one (its pointwise part gives the rows to transform).
enum RowOp : int {
  RO_NONE = 0,
  RO_RES,       // -> M_RES
  RO_RES_CG,    // M_RES -> M_CG (the first iteration of a Newton step)
  RO_CG_CG,     // M_CG -> M_CG
  RO_ASM,       // -> PF_ASM
  RO_ASM_PQ,    // PF_ASM -> PF_PQ (the first iteration)
  RO_ASM_WAIT,  // PF_ASM -> PF_WAIT
  RO_R_PQ,      // PF_R -> PF_PQ
  RO_PQ,        // -> PF_PQ (the first iteration), after PF_WAIT
  RO_PFR,       // -> PF_R
  RO_AM,        // -> AM_CHK
  RO_RESTORE,   // -> TD_RESTORE
  RO_STATS,     // -> STATS
  RO_X_IN,      // -> a diagnostic operator
  RO_X_OUT,     // a diagnostic operator -> X_END
};
__device__ __forceinline__ int row_op(int inv, int phase) {
  switch (phase) {
    case PH_M_RES: return RO_RES;
    case PH_M_CG: return inv == PH_M_RES ? RO_RES_CG : RO_CG_CG;
    case PH_PF_ASM: return RO_ASM;
    case PH_PF_PQ: return inv == PH_PF_ASM ? RO_ASM_PQ : (inv == PH_PF_R ? RO_R_PQ : RO_PQ);
    case PH_PF_WAIT: return RO_ASM_WAIT;
    case PH_PF_R: return RO_PFR;
    case PH_AM_CHK: return RO_AM;
    case PH_TD_RESTORE: return RO_RESTORE;
    case PH_STATS: return RO_STATS;
    case PH_X_PROJ:
    case PH_X_DISP:
    case PH_X_LAP: return RO_X_IN;
    case PH_X_END: return RO_X_OUT;
    default: return RO_NONE;
  }
}
// components that arrive from / leave for the column kernel
__device__ __forceinline__ constexpr int op_comps_in(int op, int inv) {
  switch (op) {
    case RO_RES_CG:
    case RO_CG_CG: return 3;
    case RO_ASM_PQ:
    case RO_ASM_WAIT:
    case RO_R_PQ: return 1;
    case RO_X_OUT: return inv == PH_X_LAP ? 1 : (inv == PH_X_DISP ? 2 : 3);
    default: return 0;
  }
}
__device__ __forceinline__ constexpr int op_comps_out(int op, int phase) {
  switch (op) {
    case RO_RES:
    case RO_RES_CG:
    case RO_CG_CG: return 3;
    case RO_R_PQ: return 2;
    case RO_ASM:
    case RO_ASM_PQ:
    case RO_PQ:
    case RO_PFR:
    case RO_STATS: return 1;
    case RO_X_IN: return phase == PH_X_LAP ? 1 : 3;
    default: return 0;
  }
}
// FP64 partial sums an op leaves for the controller (the leading entries of
// its accumulators; RP_* below), and the entry that is a maximum
__device__ __forceinline__ constexpr int op_nacc(int op) {
  switch (op) {
    case RO_RES:
    case RO_ASM: return 2;
    case RO_RES_CG:
    case RO_CG_CG: return 1;
    case RO_ASM_PQ:
    case RO_PQ: return 5;
    case RO_ASM_WAIT: return 4;
    case RO_R_PQ:
    case RO_STATS: return 8;
    case RO_AM: return 1;
    default: return 0;
  }
}
__device__ __forceinline__ constexpr int op_maxslot(int op) {
  return op == RO_STATS ? 3 : ((op == RO_ASM || op == RO_ASM_WAIT || op == RO_ASM_PQ) ? 1 : -1);
}
// M_RES: 0 ||sigma(eps_bar)||^2, 1 ||sigma||^2.  M_CG: 0 p.Cp.
// PF_ASM: 0 ||b||^2, 1 max -h'(phi_n) psi0+.
// Residual of PF_ASM / PF_R and PF_PQ (r: residual, m p: the direction on
// the inactive pixels): 0 ||r||^2, 1 r.r_old (PF_R) or max -F_phi (PF_ASM),
// 2 ||phi||^2, 3 ||d phi||^2, 4 sum d r^2, 5 sum d r mp, 6 sum d mp^2,
// 7 r.mp.

// Per-slot scalars of a tick used by the row kernels' pointwise work.
template <typename real>
struct RowCtx {
  int op, flags, split, contact, n, nin, nout;  // split: driving-force model, contact: stress model
  real lt, mt, kres, eb0, eb1, eb2, alpha_m, beta_m, beta_pf, alpha_pf;
  real ne_gamma;  // near-equilibrium strain scaling (FL_NE_SCALE)
  double eta_dt;
};

// A value that every lane holds alike (read from LDS), in scalar registers:
// the branches on it are then scalar branches.
__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ double uni(double v) { return read_lane(v, 0); }
__device__ __forceinline__ float uni(float v) { return __int_as_float(uni(__float_as_int(v))); }

template <typename real>
__device__ __forceinline__ RowCtx<real> row_ctx(const SlotCtl& ctl, const SlotParam& P, int n) {
  RowCtx<real> X;
  const int inv = uni(ctl.inv), phase = uni(ctl.phase);
  X.op = row_op(inv, phase);
  X.flags = uni(ctl.flags);
  X.split = P.split;
  X.contact = P.contact;
  X.n = n;
  X.nin = op_comps_in(X.op, inv);
  X.nout = op_comps_out(X.op, phase);
  X.lt = real(P.lam_t);
  X.mt = real(P.mu_t);
  X.kres = real(P.k_res);
  X.eb0 = uni(real(ctl.eps_bar[0]));
  X.eb1 = uni(real(ctl.eps_bar[1]));
  X.eb2 = uni(real(ctl.eps_bar[2]));
  X.alpha_m = uni(real(ctl.alpha_m));
  X.beta_m = uni(real(ctl.beta_m));
  X.beta_pf = uni(real(ctl.beta_pf));
  X.alpha_pf = uni(real(ctl.alpha_pf));
  X.eta_dt = uni(ctl.eta_dt);
  X.ne_gamma = uni(real(ctl.gamma));
  return X;
}

// Field planes of a slot, restrict-qualified through the kernel's call chain
// so that loads of later pixel pairs may be issued before stores of earlier
// ones (the pairs never overlap).
#define SPFF_PLANES                                                                                        \
  const real *__restrict__ Ep, real *__restrict__ phip, real *__restrict__ prefp, real *__restrict__ epsp, \
      real *__restrict__ thp, real *__restrict__ rmp, real *__restrict__ pmp
#define SPFF_PLANE_ARGS Ep, phip, prefp, epsp, thp, rmp, pmp

// Inputs of one pixel pair: field values and two active-set bytes.  The
// slots each op uses are those of pair_load / pair_work.
template <typename real>
struct RowIn {
  V2<real> a[11];
  unsigned short m;
};

// The CG vector updates of one pixel pair and tensor component, which need
// nothing of the other components: of the register kinds they run right
// after the component's inverse transform, so that one component's vectors
// are in registers at a time.  q: the inverse-transformed residual r;
// receives the direction p.
//   M_RES -> M_CG   p = r
//   M_CG  -> M_CG   theta += alpha p, p = r + beta p (theta = 0 before a
//                   Newton step's first iteration: FL_THETA_FIRST)
template <typename real>
struct CompIn {
  V2<real> p, th;
};
template <typename real, int OP, int NQ, int OSTEP>
__device__ __forceinline__ void comp_load(const RowCtx<real>& X, const real* __restrict__ pk,
                                          const real* __restrict__ tk, At o0, CompIn<real> (&in)[NQ]) {
  if constexpr (OP == RO_CG_CG) {
#pragma unroll
    for (int i = 0; i < NQ; ++i) in[i].p = ld2(pk, o0 + i * OSTEP);
    if (!(X.flags & FL_THETA_FIRST)) {
#pragma unroll
      for (int i = 0; i < NQ; ++i) in[i].th = ld2(tk, o0 + i * OSTEP);
    }
  }
}
template <typename real, int OP>
__device__ __forceinline__ void comp_update(const RowCtx<real>& X, real* __restrict__ pk, real* __restrict__ tk, At o,
                                            const CompIn<real>& in, cplx<real>& q) {
  using C = cplx<real>;
  if constexpr (OP == RO_CG_CG) {
    const bool first = X.flags & FL_THETA_FIRST;
    st2(tk, o, (first ? real(0) : in.th.a) + X.alpha_m * in.p.a, (first ? real(0) : in.th.b) + X.alpha_m * in.p.b);
    q = mk<C>(q.x + X.beta_m * in.p.a, q.y + X.beta_m * in.p.b);
  }
  st2(pk, o, q.x, q.y);
}

// Loads the inputs of the CH pixel pairs o0 + c OSTEP, all before any of
// them is used: the arithmetic of a pair branches (the spectral split) and
// ends in stores, and on this GPU a wait for a load also waits for the
// stores issued before it, so a pair at a time costs a memory round trip
// each.  Loads that depend on the flags are grouped under one test.
// PNEW: the direction that comp_update stored is read back (from the L2)
// rather than kept in registers.
template <typename real, int OP, int CH, int OSTEP, bool PNEW>
__device__ __forceinline__ void pair_load(const RowCtx<real>& X, SPFF_PLANES, At o0, RowIn<real> (&in)[CH]) {
  const int n = X.n, flags = X.flags;
#define SPFF_EACH(...)                  \
  _Pragma("unroll") for (int c = 0; c < CH; ++c) { \
    const At o = o0 + c * OSTEP;       \
    RowIn<real>& I = in[c];             \
    __VA_ARGS__                         \
  }
#define SPFF_LD3(S, PL) _Pragma("unroll") for (int k = 0; k < 3; ++k) I.a[(S) + k] = ld2((PL) + k * n, o);
  if constexpr (OP == RO_RES || OP == RO_RES_CG || OP == RO_CG_CG || OP == RO_ASM || OP == RO_STATS) {
    SPFF_EACH(I.a[0] = ld2(Ep, o); I.a[1] = ld2(phip, o);)
    if (OP == RO_RES || OP == RO_ASM || OP == RO_STATS || X.contact != 0) SPFF_EACH(SPFF_LD3(2, epsp))
  }
  if constexpr (OP == RO_RES) {
    if (flags & FL_THETA_PENDING) {
      if (!(flags & FL_THETA_FIRST)) SPFF_EACH(SPFF_LD3(5, thp))
      SPFF_EACH(SPFF_LD3(8, pmp))
    }
  }
  if constexpr (PNEW && (OP == RO_RES_CG || OP == RO_CG_CG)) SPFF_EACH(SPFF_LD3(8, pmp))
  if constexpr (OP == RO_ASM) SPFF_EACH(I.a[5] = ld2(prefp, o);)
  if constexpr (OP == RO_ASM_PQ || OP == RO_ASM_WAIT || OP == RO_R_PQ) {
    SPFF_EACH(I.a[0] = ld2(phip, o); I.a[1] = ld2(thp, o); I.a[2] = ld2(thp + n, o); I.a[3] = ld2(prefp, o);
              if constexpr (OP == RO_R_PQ) {
                I.a[4] = ld2(rmp, o);
                I.a[5] = ld2(pmp, o);
              })
  }
  if constexpr (OP == RO_PQ) SPFF_EACH(I.a[0] = ld2(rmp, o); I.a[1] = ld2(thp, o);)
  if constexpr (OP == RO_PFR) {
    const unsigned char* mask = reinterpret_cast<const unsigned char*>(pmp + n);
    SPFF_EACH(I.a[0] = ld2(phip, o); I.a[1] = ld2(prefp, o); I.a[2] = ld2(rmp, o);)
    if (!(flags & FL_PF_FIRST)) SPFF_EACH(I.a[3] = ld2(pmp, o); I.m = ldm<real>(mask, o);)
  }
  if constexpr (OP == RO_AM) SPFF_EACH(I.a[0] = ld2(phip, o); I.a[1] = ld2(thp + 2 * n, o);)
  if constexpr (OP == RO_RESTORE) SPFF_EACH(I.a[0] = ld2(prefp, o);)
  if constexpr (OP == RO_X_IN) SPFF_EACH(for (int k = 0; k < 3; ++k) if (k < X.nout) I.a[k] = ld2(thp + k * n, o);)
#undef SPFF_EACH
#undef SPFF_LD3
}

// The pointwise work of one pixel pair (o, o + 1): q holds the
// inverse-transformed values of the finished phase (x: o, y: o + 1; for the
// CG ops the direction p that comp_update made of them) and receives the
// values that enter the next phase's transforms.
template <typename real, int OP>
__device__ __forceinline__ void pair_work(const RowCtx<real>& X, const SlotParam& P, SPFF_PLANES, At o,
                                          const RowIn<real>& in, cplx<real> (&q)[3], double (&acc)[NP_ROW]) {
  using C = cplx<real>;
  const int n = X.n, flags = X.flags;
  [[maybe_unused]] const real eb[3] = {X.eb0, X.eb1, X.eb2};
  // two pixels of three planes as tensors
  [[maybe_unused]] auto tens = [](V2<real> x, V2<real> y, V2<real> s, int k) {
    return Sym<real>{k ? x.b : x.a, k ? y.b : y.a, k ? s.b : s.a};
  };
  [[maybe_unused]] auto el = [](V2<real> v, int k) { return k ? v.b : v.a; };
  if constexpr (OP == RO_RES) {
    V2<real> e[3] = {in.a[2], in.a[3], in.a[4]};
    if (flags & FL_FIRST_OF_STEP) st2(prefp, o, in.a[1].a, in.a[1].b);
    if (flags & FL_THETA_PENDING) {
      // the CG's last step alpha p is not in theta yet
      const bool first = flags & FL_THETA_FIRST;
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        const V2<real> to = in.a[5 + k], po = in.a[8 + k];
        const V2<real> th = {(first ? real(0) : to.a) + X.alpha_m * po.a, (first ? real(0) : to.b) + X.alpha_m * po.b};
        e[k] = {e[k].a + th.a, e[k].b + th.b};
        st2(epsp + k * n, o, e[k].a, e[k].b);
      }
    }
    // ||sigma(eps_bar)|| is the reference of a solve's first residual only
    const bool ref = !(flags & FL_MECH_STARTED);
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const real E = el(in.a[0], k), ph = el(in.a[1], k);
      const real lam = X.lt * E, mu = X.mt * E;
      const real hk = (real(1) - ph) * (real(1) - ph) + X.kres;
      const Sym<real> t = tens(e[0], e[1], e[2], k);
      const Sym<real> eps = {eb[0] + t.xx, eb[1] + t.yy, eb[2] + t.xy};
      const Sym<real> sg = stress(eps, lam, mu, hk, X.contact);
      if (ref) {
        const Sym<real> eh = {eb[0], eb[1], eb[2]};
        const Sym<real> sh = stress(eh, lam, mu, hk, X.contact);
        acc[0] += double(ddot(sh, sh));
      }
      acc[1] += double(ddot(sg, sg));
      (k ? q[0].y : q[0].x) = sg.xx;
      (k ? q[1].y : q[1].x) = sg.yy;
      (k ? q[2].y : q[2].x) = sg.xy;
    }
  }
  if constexpr (OP == RO_RES_CG || OP == RO_CG_CG) {
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const real E = el(in.a[0], k), ph = el(in.a[1], k);
      const real lam = X.lt * E, mu = X.mt * E;
      const real hk = (real(1) - ph) * (real(1) - ph) + X.kres;
      Sym<real> eps = {eb[0], eb[1], eb[2]};
      if (X.contact != 0) {
        const Sym<real> t = tens(in.a[2], in.a[3], in.a[4], k);
        eps = {eb[0] + t.xx, eb[1] + t.yy, eb[2] + t.xy};
      }
      const Sym<real> pv = {k ? q[0].y : q[0].x, k ? q[1].y : q[1].x, k ? q[2].y : q[2].x};
      const Sym<real> cp = tangent(eps, pv, lam, mu, hk, X.contact);
      acc[0] += double(ddot(pv, cp));
      (k ? q[0].y : q[0].x) = cp.xx;
      (k ? q[1].y : q[1].x) = cp.yy;
      (k ? q[2].y : q[2].x) = cp.xy;
    }
  }
  if constexpr (OP == RO_ASM) {
    V2<real> e[3] = {in.a[2], in.a[3], in.a[4]};
    if (flags & FL_NE_SCALE) {
      // near-equilibrium evolution: eps* <- gamma eps* (eps_bar was scaled
      // by the controller)
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        e[k] = {X.ne_gamma * e[k].a, X.ne_gamma * e[k].b};
        st2(epsp + k * n, o, e[k].a, e[k].b);
      }
    }
    real dv[2], bv[2], cv[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const real E = el(in.a[0], k), ph = el(in.a[1], k), rv = el(in.a[5], k);
      const real lam = X.lt * E, mu = X.mt * E;
      const Sym<real> t = tens(e[0], e[1], e[2], k);
      const Sym<real> eps = {eb[0] + t.xx, eb[1] + t.yy, eb[2] + t.xy};
      real pp, pm;
      energies(eps, lam, mu, X.split, &pp, &pm);
      dv[k] = real(2) * pp + real(P.cwl * P.wpp + X.eta_dt);
      // crack driving force -h'(phi_n) psi0+ (near-equilibrium trigger)
      if (flags & FL_NE_CHECK) acc[1] = fmax(acc[1], double(real(2) * (real(1) - rv) * pp));
      bv[k] = real(2) * pp - real(P.cwl * P.dw0) + real(X.eta_dt) * rv;
      cv[k] = fmin(fmax(ph, lower_bound(rv, P)), real(1));
      acc[0] += double(bv[k]) * double(bv[k]);
    }
    st2(thp, o, dv[0], dv[1]);
    st2(thp + n, o, bv[0], bv[1]);
    st2(thp + 2 * n, o, in.a[1].a, in.a[1].b);  // phi at the start of this PF solve
    st2(phip, o, cv[0], cv[1]);
    q[0] = mk<C>(cv[0], cv[1]);
  }
  if constexpr (OP == RO_ASM_PQ || OP == RO_ASM_WAIT || OP == RO_R_PQ) {
    const C lap = q[0];
    const V2<real> ph = in.a[0], d = in.a[1], b = in.a[2], pr = in.a[3];
    const real rr0 = d.a * ph.a + lap.x - b.a;
    const real rr1 = d.b * ph.b + lap.y - b.b;
    const real lo0 = lower_bound(pr.a, P), lo1 = lower_bound(pr.b, P);
    const bool a0 = (ph.a <= lo0 && rr0 > real(0)) || (ph.a >= real(1) && rr0 < real(0));
    const bool a1 = (ph.b <= lo1 && rr1 > real(0)) || (ph.b >= real(1) && rr1 < real(0));
    const real r0 = a0 ? real(0) : rr0, r1 = a1 ? real(0) : rr1;
    if constexpr (OP == RO_ASM_WAIT) {
      // near-equilibrium evolution: phi = phi_n here, so the unmasked
      // residual is F_phi(phi_n, eps_n); keep it for the search of x*
      st2(rmp + n, o, rr0, rr1);
      acc[1] = fmax(acc[1], fmax(-double(rr0), -double(rr1)));
    }
    st2(rmp, o, r0, r1);
    acc[0] += double(r0) * r0 + double(r1) * r1;
    acc[2] += double(ph.a) * ph.a + double(ph.b) * ph.b;
    acc[3] += double(d.a * ph.a) * double(d.a * ph.a) + double(d.b * ph.b) * double(d.b * ph.b);
    if constexpr (OP != RO_ASM_WAIT) {
      acc[4] += double(d.a) * double(r0) * double(r0) + double(d.b) * double(r1) * double(r1);
      q[0] = mk<C>(r0, r1);
    }
    if constexpr (OP == RO_R_PQ) {
      unsigned char* mask = reinterpret_cast<unsigned char*>(pmp + n);
      stm<real>(mask, o, a0, a1);
      const V2<real> ro = in.a[4];
      const real m0 = a0 ? real(0) : in.a[5].a, m1 = a1 ? real(0) : in.a[5].b;
      acc[1] += double(r0) * ro.a + double(r1) * ro.b;
      acc[5] += double(d.a) * double(r0) * double(m0) + double(d.b) * double(r1) * double(m1);
      acc[6] += double(d.a) * double(m0) * double(m0) + double(d.b) * double(m1) * double(m1);
      acc[7] += double(r0) * m0 + double(r1) * m1;
      q[1] = mk<C>(m0, m1);
    }
  }
  if constexpr (OP == RO_PQ) {
    const V2<real> r = in.a[0], d = in.a[1];
    acc[0] += double(r.a) * r.a + double(r.b) * r.b;
    acc[4] += double(d.a) * double(r.a) * double(r.a) + double(d.b) * double(r.b) * double(r.b);
    q[0] = mk<C>(r.a, r.b);
  }
  if constexpr (OP == RO_PFR) {
    const V2<real> ph = in.a[0], pr = in.a[1], r = in.a[2];
    V2<real> p = {-r.a, -r.b};
    if (!(flags & FL_PF_FIRST)) {
      p = {-r.a + X.beta_pf * in.a[3].a, -r.b + X.beta_pf * in.a[3].b};
      if (in.m & 0xffu) p.a = real(0);
      if (in.m >> 8) p.b = real(0);
    }
    st2(pmp, o, p.a, p.b);
    const real a0 = fmin(fmax(ph.a + X.alpha_pf * p.a, lower_bound(pr.a, P)), real(1));
    const real a1 = fmin(fmax(ph.b + X.alpha_pf * p.b, lower_bound(pr.b, P)), real(1));
    st2(phip, o, a0, a1);
    q[0] = mk<C>(a0, a1);
  }
  if constexpr (OP == RO_RESTORE) st2(phip, o, in.a[0].a, in.a[0].b);
  if constexpr (OP == RO_AM)
    acc[0] += fabs(double(in.a[0].a) - double(in.a[1].a)) + fabs(double(in.a[0].b) - double(in.a[1].b));
  if constexpr (OP == RO_STATS) {
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const real E = el(in.a[0], k), pv = el(in.a[1], k);
      const real lam = X.lt * E, mu = X.mt * E;
      const real hk = (real(1) - pv) * (real(1) - pv) + X.kres;
      const Sym<real> t = tens(in.a[2], in.a[3], in.a[4], k);
      const Sym<real> eps = {eb[0] + t.xx, eb[1] + t.yy, eb[2] + t.xy};
      real pp, pm;
      energies(eps, lam, mu, X.contact, &pp, &pm);  // elastic energy of the stress model
      const Sym<real> sg = stress(eps, lam, mu, hk, X.contact);
      acc[0] += double(hk) * double(pp) + double(pm);
      acc[1] += P.at == 1 ? double(pv) : double(pv) * double(pv);
      acc[2] += double(pv);
      acc[3] = fmax(acc[3], double(pv));
      acc[4] += pv > real(0.9) ? 1.0 : 0.0;
      acc[5] += double(sg.xx);
      acc[6] += double(sg.yy);
      acc[7] += double(sg.xy);
      (k ? q[0].y : q[0].x) = pv;
    }
  }
  if constexpr (OP == RO_X_IN) {
#pragma unroll
    for (int k = 0; k < 3; ++k)
      if (k < X.nout) q[k] = mk<C>(in.a[k].a, in.a[k].b);
  }
  if constexpr (OP == RO_X_OUT) {
#pragma unroll
    for (int k = 0; k < 3; ++k)
      if (k < X.nin) st2(rmp + k * n, o, q[k].x, q[k].y);
  }
}

// Makes the compiler finish the sums so far: it would otherwise put the FP64
// additions of all of a lane's pixels off to the end and keep their FP32
// terms in registers until then.
template <int NP>
__device__ __forceinline__ void settle(double (&acc)[NP], int first, int last) {
#pragma unroll
  for (int i = 0; i < NP; ++i)
    if (i >= first && i < last) asm volatile("" : "+v"(acc[i]));
}

// Calls F<op>() for the op of this tick.
#define SPFF_ROW_SWITCH(op, F) \
  switch (op) {                \
    case RO_RES: F(RO_RES); break;           \
    case RO_RES_CG: F(RO_RES_CG); break;     \
    case RO_CG_CG: F(RO_CG_CG); break;       \
    case RO_ASM: F(RO_ASM); break;           \
    case RO_ASM_PQ: F(RO_ASM_PQ); break;     \
    case RO_ASM_WAIT: F(RO_ASM_WAIT); break; \
    case RO_R_PQ: F(RO_R_PQ); break;         \
    case RO_PQ: F(RO_PQ); break;             \
    case RO_PFR: F(RO_PFR); break;           \
    case RO_AM: F(RO_AM); break;             \
    case RO_RESTORE: F(RO_RESTORE); break;   \
    case RO_STATS: F(RO_STATS); break;       \
    case RO_X_IN: F(RO_X_IN); break;         \
    case RO_X_OUT: F(RO_X_OUT); break;       \
    default: break;                          \
  }

// The pointwise work of a lane's NQ pixel pairs o0 + i OSTEP, in chunks of
// CH pairs that are loaded in full before their arithmetic.
template <typename real, int OP, int NQ, int CH, int OSTEP, bool PNEW>
__device__ __forceinline__ void row_pairs(const RowCtx<real>& X, const SlotParam& P, SPFF_PLANES, At o0,
                                          cplx<real> (&v)[3][NQ], double (&acc)[NP_ROW]) {
  static_assert(NQ % CH == 0, "pairs per lane in whole chunks");
#pragma unroll
  for (int q0 = 0; q0 < NQ; q0 += CH) {
    RowIn<real> in[CH];
    if (q0) asm volatile("" ::: "memory");  // keeps later chunks' loads out of this chunk's registers
    pair_load<real, OP, CH, OSTEP, PNEW>(X, SPFF_PLANE_ARGS, o0 + q0 * OSTEP, in);
#pragma unroll
    for (int c = 0; c < CH; ++c) {
      cplx<real> q[3];
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        if constexpr (PNEW && (OP == RO_RES_CG || OP == RO_CG_CG))
          q[k] = mk<cplx<real>>(in[c].a[8 + k].a, in[c].a[8 + k].b);
        else
          q[k] = v[k][q0 + c];
      }
      pair_work<real, OP>(X, P, SPFF_PLANE_ARGS, o0 + (q0 + c) * OSTEP, in[c], q, acc);
#pragma unroll
      for (int k = 0; k < 3; ++k) v[k][q0 + c] = q[k];
    }
    settle(acc, 0, op_nacc(OP));
  }
}

// Inputs of the controller step that a row kernel runs for the previous
// tick (and the closing kernel for the last tick of a block).
struct CtrlArgs {
  const SlotCtl* ctl_in;  // control blocks as the previous tick left them
  SlotCtl* ctl_out;       // advanced blocks, read by this tick's column kernel
  const double* prow;     // partial sums of the previous tick
  const double* pcol;
  double* prof;
  SlotSeq* seqs;
  StepRec* recs;
  unsigned long long* post;  // progress word per slot in pinned host memory, or null
  SlotCtl* mirror;           // host mirror of the control blocks (closing kernel), or null
  int ngc;
};

template <typename real>
__device__ __forceinline__ void ctrl_slot(int s, const SlotParam* __restrict__ prms, SlotCtl& C, bool writer,
                                          const double* __restrict__ prow, const double* __restrict__ pcol,
                                          double* __restrict__ prof, SlotSeq* __restrict__ seqs,
                                          StepRec* __restrict__ recs, int nx, int ny, int ngr, int ngc,
                                          const EarlyPartials& early);

// Timers of a row kernel's two parts (null when profiling is off).
struct RowTimers {
  KTime* inv;
  KTime* fwd;
};
__device__ __forceinline__ void row_middle(const RowTimers& T);

__device__ __forceinline__ void init_acc(int op, double (&acc)[NP_ROW]) {
#pragma unroll
  for (int i = 0; i < NP_ROW; ++i) acc[i] = 0.0;
  if (op == RO_STATS) acc[3] = -1.0e300;
  if (op == RO_ASM_WAIT || op == RO_ASM_PQ) acc[1] = -1.0e300;
}

// Twiddle factors of a register kind's transforms in LDS.  A global load waits for
// every load and store that its wavefront issued before it, so twiddles read
// from memory made each transform wait for the field stores ahead of it; LDS
// reads are counted apart.  The loads are issued first thing in the kernel,
// the table is stored once the control block is known.
template <typename real, int NT>
struct TwLoad {
  cplx<real> t[NT];
  __device__ __forceinline__ void load(const cplx<real>* tw, int count) {
#pragma unroll
    for (int k = 0; k < NT; ++k) {
      const int i = threadIdx.x + k * blockDim.x;
      if (i < count) t[k] = ldc<real>(tw, (unsigned)i);
    }
  }
  __device__ __forceinline__ void store(cplx<real>* tab, int count) const {
#pragma unroll
    for (int k = 0; k < NT; ++k) {
      const int i = threadIdx.x + k * blockDim.x;
      if (i < count) tab[i] = t[k];
    }
  }
};

// Control block of slot s for this tick, in `lc` (LDS): a copy of the input
// block, advanced by the controller step of the previous tick if that is
// still pending.  Every work-group of the slot computes the same block (the
// same inputs reduced in the same order); the one that owns row block 0
// (`writer`) publishes it to ctl_out and records the step.  The input block
// is not written, so groups that start late read what the early ones read.
// Every thread of the group calls this (it synchronises the group); `also`
// runs in every thread before the last synchronisation.
template <typename real, typename Also>
__device__ __forceinline__ void tick_control(int s, bool writer, const CtrlArgs& A,
                                             const SlotParam* __restrict__ prms, int nx, int ny, int ngr,
                                             SlotCtl& lc, Also also) {
  constexpr int NW = (int)(sizeof(SlotCtl) / sizeof(int));
  static_assert(sizeof(SlotCtl) % sizeof(int) == 0, "the control block is copied as words");
  const int* src = reinterpret_cast<const int*>(A.ctl_in + s);
  int* dst = reinterpret_cast<int*>(&lc);
  EarlyPartials early;
  int w[2];  // NW words by at least 64 threads
  static_assert(NW <= 128, "two words per thread hold the control block");
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const int i = threadIdx.x + k * blockDim.x;
    if (i < NW) w[k] = src[i];
  }
  if (threadIdx.x < 64)
    early.load(A.prow + (size_t)s * NP_ROW * ngr, ngr, A.pcol + (size_t)s * NP_COL * A.ngc, A.ngc);
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const int i = threadIdx.x + k * blockDim.x;
    if (i < NW) dst[i] = w[k];
  }
  __syncthreads();
  if (threadIdx.x < 64) {
    if (lc.pending)
      ctrl_slot<real>(s, prms, lc, writer, A.prow, A.pcol, A.prof, A.seqs, A.recs, nx, ny, ngr, A.ngc, early);
    // the slot's controller step after this tick is pending if it works
    if (threadIdx.x == 0) {
      lc.pending = lc.phase != PH_IDLE ? 1 : 0;
      const uint32_t no = ++lc.tick_no;
      if (lc.phase == PH_IDLE && lc.idle_at == 0) lc.idle_at = no;
      // one word, so that the host needs no ordering between two
      if (writer && A.post)
        __hip_atomic_store(A.post + s, ((unsigned long long)lc.idle_at << 32) | no, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_SYSTEM);
    }
  }
  also();
  __syncthreads();
  if (writer) {
    int* out = reinterpret_cast<int*>(A.ctl_out + s);
    for (int i = threadIdx.x; i < NW; i += blockDim.x) out[i] = dst[i];
  }
}

// ===========================================================================
// Row kernel (LDS kind): transposed load of the half spectra -> C2R row FFTs
// -> pointwise work -> R2C row FFTs -> transposed store; FP64 partial sums
// per work-group.  Each part runs if the slot's phases need it.
// ===========================================================================
template <typename real>
__device__ __forceinline__ void k_row_body(const int* __restrict__ list, const SlotPtr<real>* __restrict__ ptrs,
                                           const SlotParam* __restrict__ prms, const CtrlArgs A,
                                           const cplx<real>* __restrict__ twx, double* __restrict__ part, int nx,
                                           int ny, int R, int ngr, const RowTimers T) {
  using C = cplx<real>;
  extern __shared__ unsigned char smem_raw[];
  __shared__ double red[(THREADS / 64) * NP_ROW];
  __shared__ SlotCtl lctl;
  int g, si;
  row_coords(ngr, g, si);
  const int s = list[si];
  if (s < 0) return;
  const int M = nx >> 1, stride = M + PAD;
  C* buf = reinterpret_cast<C*>(smem_raw);
  tick_control<real>(s, g == 0, A, prms, nx, ny, ngr, lctl, []() {});
  const SlotParam& P = prms[s];
  const SlotPtr<real> F = ptrs[s];
  const int n = nx * ny;
  const RowCtx<real> X = row_ctx<real>(lctl, P, n);
  if (X.op == RO_NONE) return;
  const int y0 = g * R;
  C* spec = reinterpret_cast<C*>(F.spec);
  const int logM = ilog2(M), logR = ilog2(R);
  if (X.nin > 0) {
    const int tot = X.nin * M * R;
    for (int idx = threadIdx.x; idx < tot; idx += blockDim.x) {
      const int r = idx & (R - 1);
      const int rest = idx >> logR;
      const int kx = rest & (M - 1), c = rest >> logM;
      buf[(c * R + r) * stride + kx] = ldc<real>(spec, (unsigned)(rest * ny + y0 + r));
    }
    __syncthreads();
    c2r_pre<real>(buf, M, X.nin * R, stride, twx);
    fft_lds<real, true, MAXE>(buf, M, X.nin * R, stride, twx, 2);
  }
  row_middle(T);
  double acc[NP_ROW];
  init_acc(X.op, acc);
  const real *Ep = F.E;
  real *phip = F.phi, *prefp = F.phi_ref, *epsp = F.eps, *thp = F.theta, *rmp = F.rm, *pmp = F.pm;
#define SPFF_ROW_LOOP(OPC)                                                                       \
  for (int idx = threadIdx.x; idx < R * M; idx += blockDim.x) {                                  \
    const int r = idx >> logM, h = idx & (M - 1);                                                \
    const At o = at<real>((y0 + r) * nx + 2 * h);                                                \
    C* b = buf + r * stride + h;                                                                 \
    RowIn<real> in[1];                                                                           \
    pair_load<real, OPC, 1, 1, false>(X, SPFF_PLANE_ARGS, o, in);                                \
    C q[3];                                                                                      \
    _Pragma("unroll") for (int c = 0; c < 3; ++c) q[c] = c < X.nin ? b[c * R * stride] : mk<C>(real(0), real(0)); \
    if constexpr (OPC == RO_RES_CG || OPC == RO_CG_CG) {                                         \
      CompIn<real> ci[3][1];                                                                     \
      _Pragma("unroll") for (int c = 0; c < 3; ++c)                                              \
          comp_load<real, OPC, 1, 1>(X, pmp + c * n, thp + c * n, o, ci[c]);                     \
      _Pragma("unroll") for (int c = 0; c < 3; ++c)                                              \
          comp_update<real, OPC>(X, pmp + c * n, thp + c * n, o, ci[c][0], q[c]);                \
    }                                                                                            \
    pair_work<real, OPC>(X, P, SPFF_PLANE_ARGS, o, in[0], q, acc);                               \
    _Pragma("unroll") for (int c = 0; c < 3; ++c) if (c < X.nout) b[c * R * stride] = q[c];      \
  }
  SPFF_ROW_SWITCH(X.op, SPFF_ROW_LOOP)
#undef SPFF_ROW_LOOP
  if (X.nout > 0) {
    __syncthreads();
    fft_lds<real, false, MAXE>(buf, M, X.nout * R, stride, twx, 2);
    r2c_post<real>(buf, M, X.nout * R, stride, twx);
    // transposed store: spec[c][kx][y0 + r]
    const int tot = X.nout * M * R;
    for (int idx = threadIdx.x; idx < tot; idx += blockDim.x) {
      const int r = idx & (R - 1);
      const int rest = idx >> logR;
      const int kx = rest & (M - 1), c = rest >> logM;
      stc<real>(spec, (unsigned)(rest * ny + y0 + r), buf[(c * R + r) * stride + kx]);
    }
  }
  block_reduce_store<NP_ROW>(acc, red, part + (size_t)s * NP_ROW * ngr + g, ngr, op_nacc(X.op), op_maxslot(X.op));
}

// ===========================================================================
// Column kernel: forward column FFTs -> per-mode operator -> inverse column
// FFTs (or a Parseval reduction only).  Normalisation 1/(nx ny) is applied
// with the operator.
// ===========================================================================
template <typename real>
__device__ __forceinline__ void project3(real* a, real fx, real fy) {
  // G^:A = A - (t.A.t) t(x)t, t = (-fy, fx)/|f|; G^ = 0 at f = 0.
  const real n2 = fx * fx + fy * fy;
  if (n2 == real(0)) {
    a[0] = a[1] = a[2] = real(0);
    return;
  }
  const real inv = real(1) / n2;
  const real txx = fy * fy * inv, tyy = fx * fx * inv, txy = -fx * fy * inv;
  const real sdot = txx * a[0] + tyy * a[1] + real(2) * txy * a[2];
  a[0] -= sdot * txx;
  a[1] -= sdot * tyy;
  a[2] -= sdot * txy;
}

// Projection at one mode of an even grid.  nyq: the mode has a Nyquist
// index (ky = ny/2, or the kx = nx/2 column); its gradient component along
// that direction is already zero in (fx, fy).  With the free Nyquist
// treatment such a mode is left unconstrained (identity).
template <typename real>
__device__ __forceinline__ void project3_mode(real* a, real fx, real fy, bool nyq, int nyq_free) {
  if (nyq && nyq_free) return;
  project3(a, fx, fy);
}

// Displacement at one mode.  The strain is the unknown of the mechanics
// problem (Sec. 3.1.1); the periodic displacement u* is recovered from the
// compatible eps* by inverting eps^ = sym(i u^ (x) xi) at each mode:
//   u^ = -i [ 2 eps^ xi / |xi|^2 - xi (xi . eps^ . xi) / |xi|^4 ],
// xi = 2 pi (fx, fy) the gradient wavevector (Nyquist components zero), and
// u^ = 0 where xi = 0 (the mean, and modes that are Nyquist in every
// direction).  v[0..2] = (xx, yy, xy) in; v[0..1] = (x, y) out, v[2] = 0;
// scale carries the 1/(nx ny) of the inverse transform.
template <typename real>
__device__ __forceinline__ void disp_part(const real* a, real gx, real gy, real* u) {
  const real n2 = gx * gx + gy * gy;
  if (n2 == real(0)) {
    u[0] = u[1] = real(0);
    return;
  }
  const real inv = real(1) / n2;
  const real ex = a[0] * gx + a[2] * gy, ey = a[2] * gx + a[1] * gy;
  const real s = (gx * ex + gy * ey) * inv;
  u[0] = (real(2) * ex - gx * s) * inv;
  u[1] = (real(2) * ey - gy * s) * inv;
}

template <typename real>
__device__ __forceinline__ void disp3(cplx<real>* v, real fx, real fy, real scale) {
  using C = cplx<real>;
  const real gx = real(TWO_PI) * fx, gy = real(TWO_PI) * fy;
  const real re[3] = {v[0].x, v[1].x, v[2].x}, im[3] = {v[0].y, v[1].y, v[2].y};
  real ur[2], ui[2];
  disp_part(re, gx, gy, ur);
  disp_part(im, gx, gy, ui);
  // -i (ur + i ui) = ui - i ur
  v[0] = mk<C>(ui[0] * scale, -ur[0] * scale);
  v[1] = mk<C>(ui[1] * scale, -ur[1] * scale);
  v[2] = mk<C>(real(0), real(0));
}

// What the column kernel does for a phase.  combine: the search direction's
// spectrum is -R + beta Q, R and Q the transforms of the residual and of the
// previous direction (components 0 and 1).
enum ColMode : int {
  CM_PROJECT = 0,  // G^, for a diagnostic
  CM_LAP,          // Laplacian symbol
  CM_SUM,          // Parseval reduction of the Laplacian's quadratic form
  CM_DISP,         // displacement
  CM_RES,          // residual r^ = -G^ sigma^ and its norm
  CM_CG,           // r^ -= alpha G^ (C p)^ and its norm
};
struct ColOp {
  int ncomp, mode;
  bool combine;
};
__device__ __forceinline__ ColOp col_op(const SlotCtl& ctl) {
  switch (ctl.phase) {
    case PH_M_RES: return {3, CM_RES, false};
    case PH_M_CG: return {3, CM_CG, false};
    case PH_X_PROJ: return {3, CM_PROJECT, false};
    case PH_X_DISP: return {3, CM_DISP, false};
    case PH_X_LAP:
    case PH_PF_ASM:
    case PH_PF_R: return {1, CM_LAP, false};
    case PH_PF_PQ: return {1, CM_SUM, ctl.inv == PH_PF_R};
    case PH_STATS: return {1, CM_SUM, false};
    default: return {0, 0, false};
  }
}

// BCCG direction coefficient of Algorithm 1 from ||r||^2 and r.r_old.
__device__ __forceinline__ double bccg_beta(double r2, double rro, const SlotCtl& C) {
  return (r2 - rro) / (C.alpha_pf * C.pq);
}

// CG step length from p.Cp and ||r||^2.
__device__ __forceinline__ double cg_alpha(double pcp, double rr) {
  return (pcp > 0.0 && isfinite(pcp)) ? rr / pcp : 0.0;
}

// The coefficient of a CM_CG (alpha) or combining CM_SUM (beta) column kernel
// from this tick's row partials; the controller reduces the same partials in
// the same order and gets the same value.  load() issues the loads of the
// first 256 work-groups' partials (the first wavefront), get() returns the
// value in every thread of the group (which it synchronises).
struct ColCoef {
  double a[2][4];
  __device__ __forceinline__ void load(const double* __restrict__ pr, int ngr, bool combine) {
    if (threadIdx.x < 64) {
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        if (j == 0 || combine) {
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            const int i = threadIdx.x + 64 * k;
            a[j][k] = i < ngr ? pr[j * ngr + i] : 0.0;
          }
        }
      }
    }
  }
  __device__ __forceinline__ double get(const double* __restrict__ pr, int ngr, const SlotCtl& ctl, bool combine) {
    __shared__ double coef;
    if (threadIdx.x < 64) {
      double o[2] = {0.0, 0.0};
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        if (j == 0 || combine) {
          double v = 0.0;
#pragma unroll
          for (int k = 0; k < 4; ++k) v += a[j][k];
          for (int i = threadIdx.x + 256; i < ngr; i += 64) v += pr[j * ngr + i];
          o[j] = wave_sum(v);
        }
      }
      if (threadIdx.x == 0) coef = combine ? bccg_beta(o[0], o[1], ctl) : cg_alpha(o[0], ctl.rr);
    }
    __syncthreads();
    return coef;
  }
};

// The mechanics residual of a mode (three components a, packed or not):
// r = -a, or r - alpha a with the stored r; stores r, leaves r / n in a and
// returns r:r.  The residual lives in Fourier space (in the planes rm, laid
// out as the spectrum): its norm is known when the column kernel ends, so
// that the row kernel after it can update the direction at once, and every
// iteration's residual is compatible up to one transform's rounding (in
// real space the rounding of each update stays, its incompatible part for
// good).
template <typename real>
__device__ __forceinline__ double col_residual(cplx<real>* a, cplx<real>* rhat, unsigned at, int d, size_t plane, bool cg,
                                               real alpha, const cplx<real>* r0, real inv_n) {
  using C = cplx<real>;
  double w = 0.0;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const C r = cg ? mk<C>(r0[c].x - alpha * a[c].x, r0[c].y - alpha * a[c].y) : mk<C>(-a[c].x, -a[c].y);
    stc<real>(rhat + c * plane, at, r, d);
    w += (c == 2 ? 2.0 : 1.0) * (double(r.x) * r.x + double(r.y) * r.y);
    a[c] = cscale(r, inv_n);
  }
  return w;
}

__device__ __forceinline__ int wave_min_int(int v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v = min(v, __shfl_xor(v, off, 64));
  return v;
}

// Near-equilibrium strain scaling (Sec. 3.2.2, Algorithm 4).  fm is the
// largest -F_phi(phi_n, eps_n); the row kernel that finished the assembly kept
// the unmasked residual F_phi in rm[1] and its per-row-group maxima in
// gmax[0 .. ngr).  x* is the first pixel (row-major) where -F_phi equals fm:
// the first row group holding the maximum, then the first pixel of that
// group's rows.  With d = -h'(phi_n) psi0+ at x*, gamma^2 =
// (fphi_max - (fm - d)) / d (psi0+ is degree-two homogeneous in the strain),
// clamped at 0 and capped at 1 + deps_max / max|eps_bar|.  Returns false
// (no scaling) when x* is not found or d is not positive.  One wavefront.
template <typename real>
__device__ bool ne_gamma(const SlotPtr<real>& F, const SlotParam& P, const SlotCtl& C, double fm,
                         const double* __restrict__ gmax, int nx, int ny, int ngr, double* gamma) {
  const int lane = threadIdx.x & 63;
  int gs = ngr;
  for (int i = lane; i < ngr; i += 64)
    if (gmax[i] == fm) {
      gs = i;
      break;
    }
  gs = wave_min_int(gs);
  if (gs >= ngr) return false;
  const int n = nx * ny, rows = ny / ngr;
  const int base = gs * rows * nx, cnt = rows * nx;
  const real* fr = F.rm + n;
  int xi = n;
  for (int i = lane; i < cnt; i += 64)
    if (-double(fr[base + i]) == fm) {
      xi = base + i;
      break;
    }
  xi = wave_min_int(xi);
  if (xi >= n) return false;
  const real E = F.E[xi], ph = F.phi_ref[xi];
  const real lam = real(P.lam_t) * E, mu = real(P.mu_t) * E;
  const Sym<real> e = {real(C.eps_bar[0]) + F.eps[xi], real(C.eps_bar[1]) + F.eps[n + xi],
                       real(C.eps_bar[2]) + F.eps[2 * n + xi]};
  real pp, pm;
  energies(e, lam, mu, P.split, &pp, &pm);
  const double d = double(real(2) * (real(1) - ph) * pp);
  if (!(d > 0.0)) return false;
  double g = sqrt(fmax((P.fphi_max - (fm - d)) / d, 0.0));
  const double eb = fmax(fabs(C.eps_bar[0]), fmax(fabs(C.eps_bar[1]), fabs(C.eps_bar[2])));
  if (eb > 0.0) g = fmin(g, 1.0 + P.deps_max / eb);
  *gamma = g;
  return true;
}

// The scaling factor of a near-equilibrium check (PF_WAIT), by one wavefront
// of the column kernel of its tick, into the first column partial: -1 if the
// strain is not to be scaled.  That kernel has no other work then and writes
// no plane.  The controller step cannot evaluate it: it runs at the start of
// every row work-group, and the row kernel that it opens stores the scaled
// strain, so a group that starts after x*'s owner has stored would read
// gamma eps* and take another factor.
template <typename real>
__device__ __forceinline__ void col_ne_gamma(const SlotPtr<real>& F, const SlotParam& P, const SlotCtl& C,
                                             const double* __restrict__ pr, double* __restrict__ out, int nx, int ny,
                                             int ngr) {
  double fm = -1.0e300, gamma = -1.0;
  for (int i = threadIdx.x; i < ngr; i += 64) fm = fmax(fm, pr[ngr + i]);
  fm = wave_max(fm);
  if (fm > P.fphi_max) ne_gamma<real>(F, P, C, fm, pr + ngr, nx, ny, ngr, &gamma);
  if (threadIdx.x == 0) *out = gamma;
}

template <typename real>
__device__ __forceinline__ void k_col_body(const int* __restrict__ list, const SlotPtr<real>* __restrict__ ptrs,
                                                 const SlotParam* __restrict__ prms,
                                                 const SlotCtl* __restrict__ ctls,
                                                 const cplx<real>* __restrict__ twy,
                                                 const double* __restrict__ part_row, double* __restrict__ part,
                                                 int nx, int ny, int W, int ngr, int ngc, int nyq_free) {
  using C = cplx<real>;
  extern __shared__ unsigned char smem_raw[];
  __shared__ double red[(THREADS / 64) * NP_COL];
  const int s = list[blockIdx.y], g = blockIdx.x;
  if (s < 0) return;
  const SlotCtl& ctl = ctls[s];
  const ColOp op = col_op(ctl);
  if (op.ncomp == 0) {
    if (ctl.phase == PH_PF_WAIT && g == 0 && threadIdx.x < 64)
      col_ne_gamma<real>(ptrs[s], prms[s], ctl, part_row + (size_t)s * NP_ROW * ngr, part + (size_t)s * NP_COL * ngc,
                         nx, ny, ngr);
    return;
  }
  const int phase = ctl.phase, ncomp = op.ncomp, mode = op.mode;
  const SlotParam& P = prms[s];
  const SlotPtr<real> F = ptrs[s];
  const int M = nx >> 1, stride = ny + PAD;
  const int kx0 = g * W;
  C* buf = reinterpret_cast<C*>(smem_raw);
  C* spec = reinterpret_cast<C*>(F.spec);
  const real inv_n = real(1.0 / (double(nx) * double(ny)));
  const real two_pi = real(TWO_PI);

  // load W columns of each component
  const int tot = ncomp * W * ny;
  const int logny = ilog2(ny), logW = ilog2(W);
  const bool mech = mode == CM_RES || mode == CM_CG;
  real coef = 0;
  if (op.combine || mode == CM_CG) {
    ColCoef cc;
    cc.load(part_row + (size_t)s * NP_ROW * ngr, ngr, op.combine);
    coef = real(cc.get(part_row + (size_t)s * NP_ROW * ngr, ngr, ctl, op.combine));
  }
  C* rhat = reinterpret_cast<C*>(F.rm);
  // one mode of the mechanics residual
  auto mech_mode = [&](C* a, int kx, int ky) {
    const unsigned at = (unsigned)(kx * ny + ky);
    C r0[3];
    if (mode == CM_CG) {
#pragma unroll
      for (int c = 0; c < 3; ++c) r0[c] = ldc<real>(rhat + (size_t)c * M * ny, at);
    }
    return col_residual<real>(a, rhat, at, 0, (size_t)M * ny, mode == CM_CG, coef, r0, inv_n);
  };
  for (int idx = threadIdx.x; idx < tot; idx += blockDim.x) {
    const int y = idx & (ny - 1), rest = idx >> logny;
    const int w = rest & (W - 1), c = rest >> logW;
    const unsigned at = (unsigned)((c * M + kx0 + w) * ny + y);
    C z = ldc<real>(spec, at);
    if (op.combine) {
      const C zq = ldc<real>(spec + (size_t)M * ny, at);
      z = mk<C>(coef * zq.x - z.x, coef * zq.y - z.y);
    }
    buf[rest * stride + y] = z;
  }
  __syncthreads();
  fft_lds<real, false, MAXE>(buf, ny, ncomp * W, stride, twy, 1);

  double acc[NP_COL] = {0.0, 0.0};
  const real lap_scale = (phase == PH_X_LAP ? real(1) : real(P.kappa)) * inv_n;
  // per-mode operator; thread owns mode (w, ky); for the packed column kx = 0
  // threads with ky <= ny/2 own the pair (ky, ny - ky)
  for (int idx = threadIdx.x; idx < W * ny; idx += blockDim.x) {
    const int w = idx >> logny, ky = idx & (ny - 1);
    const int kx = kx0 + w;
    const int kys = ky < ny / 2 ? ky : ky - ny;
    const real fy_true = real(kys) / real(ny);
    const real fy_grad = (2 * ky == ny) ? real(0) : fy_true;
    if (kx > 0) {
      const real fx = real(kx) / real(nx);
      if (mode == CM_DISP) {
        C a[3] = {buf[(0 * W + w) * stride + ky], buf[(1 * W + w) * stride + ky], buf[(2 * W + w) * stride + ky]};
        disp3(a, fx, fy_grad, inv_n);
#pragma unroll
        for (int c = 0; c < 3; ++c) buf[(c * W + w) * stride + ky] = a[c];
      } else if (mode == CM_PROJECT || mech) {
        C* a0 = buf + (0 * W + w) * stride + ky;
        C* a1 = buf + (1 * W + w) * stride + ky;
        C* a2 = buf + (2 * W + w) * stride + ky;
        real re[3] = {a0->x, a1->x, a2->x}, im[3] = {a0->y, a1->y, a2->y};
        project3_mode(re, fx, fy_grad, 2 * ky == ny, nyq_free);
        project3_mode(im, fx, fy_grad, 2 * ky == ny, nyq_free);
        if (mech) {
          C a[3] = {mk<C>(re[0], im[0]), mk<C>(re[1], im[1]), mk<C>(re[2], im[2])};
          acc[0] += 2.0 * mech_mode(a, kx, ky);
          *a0 = a[0];
          *a1 = a[1];
          *a2 = a[2];
        } else {
          *a0 = mk<C>(re[0] * inv_n, im[0] * inv_n);
          *a1 = mk<C>(re[1] * inv_n, im[1] * inv_n);
          *a2 = mk<C>(re[2] * inv_n, im[2] * inv_n);
        }
      } else {
        const real L = two_pi * two_pi * (fx * fx + fy_true * fy_true);
        C* a = buf + w * stride + ky;
        if (mode == CM_LAP) {
          *a = cscale(*a, L * lap_scale);
        } else {
          const C v = *a;
          acc[0] += 2.0 * double(L) * (double(v.x) * double(v.x) + double(v.y) * double(v.y));
        }
      }
    } else {
      if (2 * ky > ny) continue;  // partner handled by ky' = ny - ky
      const int km = (ny - ky) & (ny - 1);
      const bool self = (km == ky);
      // split packed column into A (kx = 0 column) and B (kx = nx/2 column)
      const real fxN_true = real(0.5);
      if (mode == CM_DISP) {
        C Aa[3], Bb[3];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          const C cp = buf[(c * W + w) * stride + ky];
          const C cm = cconj(buf[(c * W + w) * stride + km]);
          Aa[c] = cscale(cadd(cp, cm), real(0.5));
          Bb[c] = cscale(cmulni(csub(cp, cm)), real(0.5));
        }
        // kx = 0 and kx = nx/2 (x-component of the gradient wavevector zero)
        disp3(Aa, real(0), fy_grad, inv_n);
        disp3(Bb, real(0), fy_grad, inv_n);
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          buf[(c * W + w) * stride + ky] = cadd(Aa[c], cmuli(Bb[c]));
          if (!self) buf[(c * W + w) * stride + km] = cadd(cconj(Aa[c]), cmuli(cconj(Bb[c])));
        }
      } else if (mode == CM_PROJECT || mech) {
        C Aa[3], Bb[3];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          const C cp = buf[(c * W + w) * stride + ky];
          const C cm = cconj(buf[(c * W + w) * stride + km]);
          Aa[c] = cscale(cadd(cp, cm), real(0.5));
          Bb[c] = cscale(cmulni(csub(cp, cm)), real(0.5));
        }
        real ar[3] = {Aa[0].x, Aa[1].x, Aa[2].x}, ai[3] = {Aa[0].y, Aa[1].y, Aa[2].y};
        real br[3] = {Bb[0].x, Bb[1].x, Bb[2].x}, bi[3] = {Bb[0].y, Bb[1].y, Bb[2].y};
        project3_mode(ar, real(0), fy_grad, 2 * ky == ny, nyq_free);
        project3_mode(ai, real(0), fy_grad, 2 * ky == ny, nyq_free);
        // kx = nx/2: gradient wavevector x-component is zero (Nyquist)
        project3_mode(br, real(0), fy_grad, true, nyq_free);
        project3_mode(bi, real(0), fy_grad, true, nyq_free);
        C zp[3], zm[3];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          const C A = mk<C>(ar[c], ai[c]), B = mk<C>(br[c], bi[c]);
          zp[c] = cadd(A, cmuli(B));
          zm[c] = cadd(cconj(A), cmuli(cconj(B)));
        }
        if (mech) {
          // the packed column's norm is that of its two halves (the cross
          // terms of Hermitian A and B cancel over +-ky)
          acc[0] += mech_mode(zp, 0, ky);
          if (!self) acc[0] += mech_mode(zm, 0, km);
        } else {
#pragma unroll
          for (int c = 0; c < 3; ++c) {
            zp[c] = cscale(zp[c], inv_n);
            zm[c] = cscale(zm[c], inv_n);
          }
        }
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          buf[(c * W + w) * stride + ky] = zp[c];
          if (!self) buf[(c * W + w) * stride + km] = zm[c];
        }
      } else {
        const C cp = buf[w * stride + ky];
        const C cm = cconj(buf[w * stride + km]);
        const C A = cscale(cadd(cp, cm), real(0.5));
        const C B = cscale(cmulni(csub(cp, cm)), real(0.5));
        const real L0 = two_pi * two_pi * (fy_true * fy_true);
        const real LN = two_pi * two_pi * (fxN_true * fxN_true + fy_true * fy_true);
        if (mode == CM_LAP) {
          const C A2 = cscale(A, L0 * lap_scale), B2 = cscale(B, LN * lap_scale);
          buf[w * stride + ky] = cadd(A2, cmuli(B2));
          if (!self) buf[w * stride + km] = cadd(cconj(A2), cmuli(cconj(B2)));
        } else {
          const double wgt = self ? 1.0 : 2.0;
          acc[0] += wgt * (double(L0) * (double(A.x) * double(A.x) + double(A.y) * double(A.y)) +
                           double(LN) * (double(B.x) * double(B.x) + double(B.y) * double(B.y)));
        }
      }
    }
  }
  __syncthreads();
  if (mode != CM_SUM) {
    fft_lds<real, true, MAXE>(buf, ny, ncomp * W, stride, twy, 1);
    for (int idx = threadIdx.x; idx < tot; idx += blockDim.x) {
      const int y = idx & (ny - 1), rest = idx >> logny;
      const int w = rest & (W - 1), c = rest >> logW;
      stc<real>(spec, (unsigned)((c * M + kx0 + w) * ny + y), buf[rest * stride + y]);
    }
  }
  block_reduce_store<NP_COL>(acc, red, part + (size_t)s * NP_COL * ngc + g, ngc, (mech || mode == CM_SUM) ? 1 : 0);
}

// Column kernel with register-resident transforms (ny = N in {128, ...,
// 2048}, FP32 and FP64; 16 points per lane FP32 only): a group of L = N/E lanes owns one kx column of every
// component, E modes per lane per component (lane l: ky = l + m L).
// Forward FFTs, the per-mode operator and the inverse FFTs run on the lane's
// registers; only the Stockham exchanges between radix-8 passes go through
// LDS, inside the group.  The packed column kx = 0 (X[0] + i X[nx/2]) takes
// the partner mode -ky from lane (L - l) mod L by a cross-lane shuffle
// (through LDS where the group spans several wavefronts).
template <typename real, int N, int E, bool AHEAD>
__device__ __forceinline__ void k_colr_body(const int* __restrict__ list, const SlotPtr<real>* __restrict__ ptrs,
                                            const SlotParam* __restrict__ prms, const SlotCtl* __restrict__ ctls,
                                            const cplx<real>* __restrict__ twy, const double* __restrict__ part_row,
                                            double* __restrict__ part, int nx, int ngr, int ngc, int nyq_free) {
  using C = cplx<real>;
  // E = 8 points per lane up to 512-point columns; 1024 and 2048 points
  // take 16 (one or two wavefronts per column) or 8 (two or four: twice
  // the wavefronts in flight for launches with one or two problems).  A
  // group wider than a wavefront is the work-group's only column, so every
  // barrier below is reached by all its threads.
  constexpr int L = N / E;
  static_assert(E == 8 || E == 16, "8 or 16 points per lane");
  static_assert(L <= 64 || N >= 1024, "groups wider than a wavefront are 1024- or 2048-point columns");
  extern __shared__ unsigned char smem_raw[];
  __shared__ double red[(THREADS / 64) * NP_COL];
  TwLoad<real, (N / 2 + 63) / 64> tl;
  tl.load(twy, N / 2);
  const int s = list[blockIdx.y], g = blockIdx.x;
  if (s < 0) return;
  const SlotCtl& ctl = ctls[s];
  const ColOp op = col_op(ctl);
  if (op.ncomp == 0) {
    if (ctl.phase == PH_PF_WAIT && g == 0 && threadIdx.x < 64)
      col_ne_gamma<real>(ptrs[s], prms[s], ctl, part_row + (size_t)s * NP_ROW * ngr, part + (size_t)s * NP_COL * ngc,
                         nx, N, ngr);
    return;
  }
  const int phase = ctl.phase, ncomp = op.ncomp, mode = op.mode;
  const SlotParam& P = prms[s];
  const SlotPtr<real> F = ptrs[s];
  const int M = nx >> 1;
  const int W = blockDim.x / L;
  C* tw = reinterpret_cast<C*>(smem_raw) + W * XArea<N>::size;
  tl.store(tw, N / 2);
  const int col = threadIdx.x / L, lane = threadIdx.x & (L - 1);
  const int kx = g * W + col;
  const unsigned at = (unsigned)(kx * N + lane);
  C* x = reinterpret_cast<C*>(smem_raw) + col * XArea<N>::size;
  C* spec = reinterpret_cast<C*>(F.spec);
  const real inv_n = real(1.0 / (double(nx) * double(N)));
  const real two_pi = real(TWO_PI);
  const real lap_scale = (phase == PH_X_LAP ? real(1) : real(P.kappa)) * inv_n;

  C v[3][E];
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    if (c < ncomp) {
#pragma unroll
      for (int m = 0; m < E; ++m) v[c][m] = ldc<real>(spec + (size_t)c * M * N, at, m * L);
    }
  }
  if (op.combine) {
#pragma unroll
    for (int m = 0; m < E; ++m) v[1][m] = ldc<real>(spec + (size_t)M * N, at, m * L);
  }
  const bool mech = mode == CM_RES || mode == CM_CG;
  real coef = 0;
  ColCoef cc;
  const double* pr = part_row + (size_t)s * NP_ROW * ngr;
  if (op.combine || mode == CM_CG) cc.load(pr, ngr, op.combine);
  C* rhat = reinterpret_cast<C*>(F.rm);
  // The stored residual.  AHEAD (launches of few wavefronts): that of the
  // first half of the modes is loaded before the transforms, the rest after
  // them, all before the first store: one memory round trip less, at a
  // wavefront per SIMD less.  Otherwise four modes at a time.
  constexpr int HR = AHEAD ? E / 2 : 0;
  C r0[3][E];
  if (AHEAD && mode == CM_CG) {
#pragma unroll
    for (int c = 0; c < 3; ++c)
#pragma unroll
      for (int m = 0; m < HR; ++m) r0[c][m] = ldc<real>(rhat + (size_t)c * M * N, at, m * L);
  }
  if (op.combine) {
    coef = real(cc.get(pr, ngr, ctl, true));
#pragma unroll
    for (int m = 0; m < E; ++m) v[0][m] = mk<C>(coef * v[1][m].x - v[0][m].x, coef * v[1][m].y - v[0][m].y);
  }
  __syncthreads();  // the twiddle table
#pragma unroll
  for (int c = 0; c < 3; ++c)
    if (c < ncomp) reg_fft<real, false, N, E>(v[c], x, lane, tw, 1);
  if (mode == CM_CG) {
    if constexpr (AHEAD) {
#pragma unroll
      for (int c = 0; c < 3; ++c)
#pragma unroll
        for (int m = HR; m < E; ++m) r0[c][m] = ldc<real>(rhat + (size_t)c * M * N, at, m * L);
    }
    coef = real(cc.get(pr, ngr, ctl, false));
  }

  double acc[NP_COL] = {0.0, 0.0};
  if (kx > 0) {
    const real fx = real(kx) / real(nx);
#pragma unroll
    for (int m = 0; m < E; ++m) {
      const int ky = lane + m * L;
      const int kys = ky < N / 2 ? ky : ky - N;
      const real fy_true = real(kys) / real(N);
      const real fy_grad = (2 * ky == N) ? real(0) : fy_true;
      if (mode == CM_DISP) {
        C a[3] = {v[0][m], v[1][m], v[2][m]};
        disp3(a, fx, fy_grad, inv_n);
#pragma unroll
        for (int c = 0; c < 3; ++c) v[c][m] = a[c];
      } else if (mode == CM_PROJECT || mech) {
        real re[3] = {v[0][m].x, v[1][m].x, v[2][m].x}, im[3] = {v[0][m].y, v[1][m].y, v[2][m].y};
        project3_mode(re, fx, fy_grad, 2 * ky == N, nyq_free);
        project3_mode(im, fx, fy_grad, 2 * ky == N, nyq_free);
#pragma unroll
        for (int c = 0; c < 3; ++c) v[c][m] = mk<C>(re[c], im[c]);
      } else {
        const real Lk = two_pi * two_pi * (fx * fx + fy_true * fy_true);
        if (mode == CM_LAP) {
          v[0][m] = cscale(v[0][m], Lk * lap_scale);
        } else {
          acc[0] += 2.0 * double(Lk) * (double(v[0][m].x) * double(v[0][m].x) + double(v[0][m].y) * double(v[0][m].y));
        }
      }
    }
  } else {
    // packed column: A = X(kx = 0), B = X(kx = nx/2) at ky, from Z(ky) and
    // conj Z(-ky); the partner of slot m of lane l is slot E-1-m of lane
    // L-l (l > 0), or slot (E-m) mod E of lane 0 itself
    C Pn[3][E];
    const int src = (L - lane) & (L - 1);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      if (c < ncomp) {
        if constexpr (L <= 64) {
#pragma unroll
          for (int i = 0; i < E; ++i) {
            const real px = __shfl(v[c][i].x, src, L), py = __shfl(v[c][i].y, src, L);
            Pn[c][E - 1 - i] = mk<C>(px, py);
          }
        } else {
          // the partner lane may sit in the other wavefront: exchange
          // through the column's LDS area (free between transforms)
#pragma unroll
          for (int i = 0; i < E; ++i) x[xpad(lane) + i * (L + L / 8)] = v[c][i];
          group_sync<L>();
#pragma unroll
          for (int i = 0; i < E; ++i) Pn[c][E - 1 - i] = x[xpad(src) + i * (L + L / 8)];
          group_sync<L>();
        }
        if (lane == 0) {
#pragma unroll
          for (int m = 0; m < E; ++m) Pn[c][m] = v[c][(E - m) & (E - 1)];
        }
      }
    }
#pragma unroll
    for (int m = 0; m < E; ++m) {
      const int ky = lane + m * L;
      const int kys = ky < N / 2 ? ky : ky - N;
      const real fy_true = real(kys) / real(N);
      const real fy_grad = (2 * ky == N) ? real(0) : fy_true;
      if (mode == CM_DISP) {
        C Aa[3], Bb[3];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          const C cp = v[c][m], cm = cconj(Pn[c][m]);
          Aa[c] = cscale(cadd(cp, cm), real(0.5));
          Bb[c] = cscale(cmulni(csub(cp, cm)), real(0.5));
        }
        disp3(Aa, real(0), fy_grad, inv_n);
        disp3(Bb, real(0), fy_grad, inv_n);
#pragma unroll
        for (int c = 0; c < 3; ++c) v[c][m] = cadd(Aa[c], cmuli(Bb[c]));
      } else if (mode == CM_PROJECT || mech) {
        real ar[3], ai[3], br[3], bi[3];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          const C cp = v[c][m], cm = cconj(Pn[c][m]);
          const C A = cscale(cadd(cp, cm), real(0.5));
          const C Bq = cscale(cmulni(csub(cp, cm)), real(0.5));
          ar[c] = A.x;
          ai[c] = A.y;
          br[c] = Bq.x;
          bi[c] = Bq.y;
        }
        project3_mode(ar, real(0), fy_grad, 2 * ky == N, nyq_free);
        project3_mode(ai, real(0), fy_grad, 2 * ky == N, nyq_free);
        // kx = nx/2: gradient wavevector x-component is zero (Nyquist)
        project3_mode(br, real(0), fy_grad, true, nyq_free);
        project3_mode(bi, real(0), fy_grad, true, nyq_free);
#pragma unroll
        for (int c = 0; c < 3; ++c) v[c][m] = cadd(mk<C>(ar[c], ai[c]), cmuli(mk<C>(br[c], bi[c])));
      } else {
        const C cp = v[0][m], cm = cconj(Pn[0][m]);
        const C A = cscale(cadd(cp, cm), real(0.5));
        const C Bq = cscale(cmulni(csub(cp, cm)), real(0.5));
        const real L0 = two_pi * two_pi * (fy_true * fy_true);
        const real LN = two_pi * two_pi * (real(0.25) + fy_true * fy_true);
        if (mode == CM_LAP) {
          v[0][m] = cadd(cscale(A, L0 * lap_scale), cmuli(cscale(Bq, LN * lap_scale)));
        } else {
          acc[0] += double(L0) * (double(A.x) * double(A.x) + double(A.y) * double(A.y)) +
                    double(LN) * (double(Bq.x) * double(Bq.x) + double(Bq.y) * double(Bq.y));
        }
      }
    }
  }
  if (mech) {
    // (a packed column's norm is that of its two halves: the cross terms of
    // the Hermitian A and B cancel over +-ky)
    const double w = kx > 0 ? 2.0 : 1.0;
#pragma unroll
    for (int m = 0; m < E; ++m) {
      if (!AHEAD && mode == CM_CG && m % 4 == 0) {
#pragma unroll
        for (int i = m; i < m + 4; ++i)
#pragma unroll
          for (int c = 0; c < 3; ++c) r0[c][i] = ldc<real>(rhat + (size_t)c * M * N, at, i * L);
      }
      C a[3] = {v[0][m], v[1][m], v[2][m]};
      const C r[3] = {r0[0][m], r0[1][m], r0[2][m]};
      acc[0] += w * col_residual<real>(a, rhat, at, m * L, (size_t)M * N, mode == CM_CG, coef, r, inv_n);
#pragma unroll
      for (int c = 0; c < 3; ++c) v[c][m] = a[c];
      if (m % 4 == 3) settle(acc, 0, 1);
    }
  } else if (mode == CM_PROJECT) {
#pragma unroll
    for (int c = 0; c < 3; ++c)
#pragma unroll
      for (int m = 0; m < E; ++m) v[c][m] = cscale(v[c][m], inv_n);
  }
  if (mode != CM_SUM) {
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      if (c < ncomp) {
        reg_fft<real, true, N, E>(v[c], x, lane, tw, 1);
#pragma unroll
        for (int m = 0; m < E; ++m) stc<real>(spec + (size_t)c * M * N, at, v[c][m], m * L);
      }
    }
  }
  block_reduce_store<NP_COL>(acc, red, part + (size_t)s * NP_COL * ngc + g, ngc, (mech || mode == CM_SUM) ? 1 : 0);
}

// ---------------------------------------------------------------------------
// Row kernel with register-resident transforms (M = nx/2 in {64 .. 1024},
// FP64 to 512): a group of L = M/E lanes (E = 4, 8, or 16 for M = 1024) owns one row
// (R = blockDim/L rows per work-group); lane l holds z[h] = x[2h] + i x[2h+1]
// for h = l + m L.  The pointwise work runs per pixel pair on the registers
// between the inverse and the forward transform; the real <-> half-spectrum
// step pairs bin k with M - k by a cross-lane shuffle (same pattern as the
// packed column); the transposed spectrum load / store goes through an LDS
// tile [kx][row] so that R consecutive y of one kx move as one run.
// ---------------------------------------------------------------------------
template <typename real, int M, int E = 8>
struct RowLds {
  // exchange areas of the R row groups, then the [kx][row] tile, then the
  // twiddle table.  FP32 rows with four points per lane hold areas and tiles
  // of all three components.  Rows of 8 KB (1024 points, 512 in FP64) let the
  // tile overlie the exchange areas (a barrier more per component): 49 KB for
  // four rows instead of 86 KB, so that a CU holds more than one work-group.
  static constexpr bool ALIAS = M * sizeof(cplx<real>) >= 8192;
  static constexpr int NC = E == 4 && sizeof(real) == 4 ? 3 : 1;
  static __device__ __forceinline__ int tile_index(int k, int r, int R) { return k * (R + 1) + r; }
  static __device__ __forceinline__ int tile(int R) { return ALIAS ? 0 : NC * R * XArea<M>::size; }
  static __device__ __forceinline__ int table(int R) {
    const int x = R * XArea<M>::size, t = M * (R + 1);
    return ALIAS ? (x > t ? x : t) : NC * (x + t);
  }
};

// partner slots for bin k = l + m L and M - k: slot E-1-m of lane L-l, or
// for lane 0 its own slot (E-m) mod E
template <typename real, int E, int L>
__device__ __forceinline__ void partner_bins(const cplx<real> (&v)[E], cplx<real> (&pn)[E], int lane) {
  const int src = (L - lane) & (L - 1);
#pragma unroll
  for (int i = 0; i < E; ++i) {
    const real px = __shfl(v[i].x, src, L), py = __shfl(v[i].y, src, L);
    pn[E - 1 - i] = mk<cplx<real>>(px, py);
  }
  if (lane == 0) {
#pragma unroll
    for (int m = 0; m < E; ++m) pn[m] = v[(E - m) & (E - 1)];
  }
}

// From a row's packed half spectrum (bin k = lane + m L; bin 0 holds X[0] + i
// X[M]) to Z whose unnormalised inverse transform gives nx (x[2h] +
// i x[2h+1]), in place; and from the transform of a real row to its half
// spectrum.
template <typename real, int M, int E>
__device__ __forceinline__ void c2r_bins(cplx<real> (&v)[E], const cplx<real>* tw, int lane) {
  using C = cplx<real>;
  constexpr int L = M / E;
  C pn[E];
  partner_bins<real, E, L>(v, pn, lane);
#pragma unroll
  for (int m = 0; m < E; ++m) {
    const int k = lane + m * L;
    if (k == 0) {
      v[m] = mk<C>(v[m].x + v[m].y, v[m].x - v[m].y);
    } else {
      const C xk = v[m], xm = cconj(pn[m]);
      const C a = cadd(xk, xm), b = csub(xk, xm);
      v[m] = cadd(a, cmuli(cmul(cconj(tw[k]), b)));
    }
  }
}
template <typename real, int M, int E>
__device__ __forceinline__ void r2c_bins(const cplx<real> (&v)[E], cplx<real> (&out)[E], const cplx<real>* tw,
                                         int lane) {
  using C = cplx<real>;
  constexpr int L = M / E;
  C pn[E];
  partner_bins<real, E, L>(v, pn, lane);
#pragma unroll
  for (int m = 0; m < E; ++m) {
    const int k = lane + m * L;
    if (k == 0) {
      out[m] = mk<C>(v[m].x + v[m].y, v[m].x - v[m].y);
    } else {
      const C zk = v[m], zm = cconj(pn[m]);
      const C e = cscale(cadd(zk, zm), real(0.5));
      const C od = cscale(cmulni(csub(zk, zm)), real(0.5));
      out[m] = cadd(e, cmul(tw[k], od));
    }
  }
}

// comp_update for a lane's pixel pairs of component c; in: their inputs,
// where they are loaded already (PRE).
template <typename real, int OP, int NQ, int OSTEP, bool PRE>
__device__ __forceinline__ void row_comp(const RowCtx<real>& X, const SlotPtr<real>& F, int c, At o0,
                                         const CompIn<real> (&pre)[NQ], cplx<real> (&v)[NQ]) {
  real *pk = F.pm + c * X.n, *tk = F.theta + c * X.n;
  constexpr int CH = NQ > 8 ? 8 : NQ;
#pragma unroll
  for (int i0 = 0; i0 < NQ; i0 += CH) {
    CompIn<real> in[CH];
    if constexpr (PRE) {
#pragma unroll
      for (int i = 0; i < CH; ++i) in[i] = pre[i0 + i];
    } else {
      if (i0) asm volatile("" ::: "memory");
      comp_load<real, OP, CH, OSTEP>(X, pk, tk, o0 + i0 * OSTEP, in);
    }
#pragma unroll
    for (int i = 0; i < CH; ++i) comp_update<real, OP>(X, pk, tk, o0 + (i0 + i) * OSTEP, in[i], v[i0 + i]);
  }
}

template <typename real, int M, int E>
__device__ __forceinline__ void k_rowr_body(const int* __restrict__ list, const SlotPtr<real>* __restrict__ ptrs,
                                            const SlotParam* __restrict__ prms, const CtrlArgs A,
                                            const cplx<real>* __restrict__ twx, double* __restrict__ part, int ny,
                                            int ngr, const RowTimers T) {
  using C = cplx<real>;
  constexpr int L = M / E, nx = 2 * M;
  extern __shared__ unsigned char smem_raw[];
  __shared__ double red[(THREADS / 64) * NP_ROW];
  __shared__ SlotCtl lctl;
  int g, si;
  row_coords(ngr, g, si);
  const int s = list[si];
  if (s < 0) return;
  const int R = blockDim.x / L, logR = ilog2(R);
  C* tile = reinterpret_cast<C*>(smem_raw) + RowLds<real, M, E>::tile(R);
  C* tw = reinterpret_cast<C*>(smem_raw) + RowLds<real, M, E>::table(R);
  const int tsize = M * (R + 1);
  TwLoad<real, M / 64> tl;
  tl.load(twx, M);
  const SlotPtr<real> F = ptrs[s];
  const SlotParam& P = prms[s];
  tick_control<real>(s, g == 0, A, prms, nx, ny, ngr, lctl, [&]() { tl.store(tw, M); });
  const int n = nx * ny;
  const RowCtx<real> X = row_ctx<real>(lctl, P, n);
  if (X.op == RO_NONE) return;
  const int row = threadIdx.x / L, lane = threadIdx.x & (L - 1);
  const int y0 = g * R;
  C* xa = reinterpret_cast<C*>(smem_raw) + row * XArea<M>::size;
  C* spec = reinterpret_cast<C*>(F.spec);

  const At o0 = at<real>((y0 + row) * nx + 2 * lane);
  // Each op has its own copy of the whole pass: values that merge before or
  // after a switch over the ops cost a wavefront per SIMD (176 registers a
  // lane instead of 138 for eight points per lane).
  auto pass = [&](auto opc) {
    constexpr int OP = decltype(opc)::value;
    constexpr bool CG = OP == RO_RES_CG || OP == RO_CG_CG;
    // a diagnostic operator's component count is known at run time
    constexpr int NIN = op_comps_in(OP, PH_X_PROJ), NOUT = op_comps_out(OP, PH_X_PROJ);
    C v[3][E];
    double acc[NP_ROW];
    init_acc(OP, acc);
    // Four points per lane is the kernel of few wavefronts: it loads the tile
    // entries of every component up front (E per thread and component: R rows
    // x M bins over R L threads) and, in FP32, takes the three transforms
    // through their passes together (ILV), which pays each memory round trip,
    // exchange and barrier once instead of three times: 11.4 -> 10.6 us a CG
    // tick at 1 x 256^2, 18.3 -> 17.7 at 13 x 256^2, 13.5 -> 12.7 at 1 x 512^2.
    // (Loading the pixel fields ahead of the transforms too gave 0.2 us at one
    // problem and took 0.4 at three: more loads in flight than the CU queues.)
    // Up to eight points per lane load a component's CG vectors before its
    // transform.
    constexpr int CH = E == 4 ? 4 : 2;
    constexpr bool ILV = E == 4 && std::is_same<real, float>::value, PREC = E <= 8;
    CompIn<real> ci[3][E];
    if constexpr (E == 4) {
#pragma unroll
      for (int c = 0; c < NIN; ++c) {
        if (OP == RO_X_OUT && c >= X.nin) break;
#pragma unroll
        for (int i = 0; i < E; ++i) {
          const int idx = threadIdx.x + i * blockDim.x;
          const int r = idx & (R - 1), k = idx >> logR;
          v[c][i] = ldc<real>(spec + (size_t)c * M * ny, (unsigned)(k * ny + y0 + r));
        }
      }
    }
    if constexpr (ILV && NIN > 0) {
      // every component at once, through tiles and exchange areas of its own
#pragma unroll
      for (int c = 0; c < NIN; ++c)
#pragma unroll
        for (int i = 0; i < E; ++i) {
          const int idx = threadIdx.x + i * blockDim.x;
          const int r = idx & (R - 1), k = idx >> logR;
          tile[c * tsize + RowLds<real, M>::tile_index(k, r, R)] = v[c][i];
        }
      __syncthreads();
#pragma unroll
      for (int c = 0; c < NIN; ++c) {
#pragma unroll
        for (int m = 0; m < E; ++m) v[c][m] = tile[c * tsize + RowLds<real, M>::tile_index(lane + m * L, row, R)];
        c2r_bins<real, M, E>(v[c], tw, lane);
      }
      if constexpr (CG) {
#pragma unroll
        for (int c = 0; c < 3; ++c) comp_load<real, OP, E, 2 * L>(X, F.pm + c * n, F.theta + c * n, o0, ci[c]);
      }
      reg_fft_n<real, true, M, E, NIN>(v, xa, R * XArea<M>::size, lane, tw, 2);
      if constexpr (CG) {
#pragma unroll
        for (int c = 0; c < 3; ++c) row_comp<real, OP, E, 2 * L, true>(X, F, c, o0, ci[c], v[c]);
      }
    } else {
#pragma unroll
    for (int c = 0; c < NIN; ++c) {
      if (OP == RO_X_OUT && c >= X.nin) break;
      if (c > 0) __syncthreads();  // the previous component's tile reads are done
      const int tid = opaque(threadIdx.x), lane = tid & (L - 1);
      if constexpr (E == 4) {
#pragma unroll
        for (int i = 0; i < E; ++i) {
          const int idx = tid + i * blockDim.x;
          const int r = idx & (R - 1), k = idx >> logR;
          tile[RowLds<real, M>::tile_index(k, r, R)] = v[c][i];
        }
      } else {
        for (int idx = tid; idx < M * R; idx += blockDim.x) {
          const int r = idx & (R - 1), k = idx >> logR;
          tile[RowLds<real, M>::tile_index(k, r, R)] =
              ldc<real>(spec + (size_t)c * M * ny, (unsigned)(k * ny + y0 + r));
        }
      }
      __syncthreads();
#pragma unroll
      for (int m = 0; m < E; ++m) v[c][m] = tile[RowLds<real, M>::tile_index(lane + m * L, row, R)];
      if constexpr (RowLds<real, M>::ALIAS) __syncthreads();
      c2r_bins<real, M, E>(v[c], tw, lane);
      if constexpr (CG && PREC)
        comp_load<real, OP, E, 2 * L>(X, F.pm + c * n, F.theta + c * n, o0, ci[c]);
      reg_fft<real, true, M, E>(v[c], xa, lane, tw, 2);
      if constexpr (CG) row_comp<real, OP, E, 2 * L, PREC>(X, F, c, o0, ci[c], v[c]);
    }
    }
    row_middle(T);
    row_pairs<real, OP, E, CH, 2 * L, E == 16>(X, P, F.E, F.phi, F.phi_ref, F.eps, F.theta, F.rm, F.pm, o0, v, acc);
    if constexpr (ILV && NOUT > 0) {
      reg_fft_n<real, false, M, E, NOUT>(v, xa, R * XArea<M>::size, lane, tw, 2);
      __syncthreads();  // the tiles are free
#pragma unroll
      for (int c = 0; c < NOUT; ++c) {
        C out[E];
        r2c_bins<real, M, E>(v[c], out, tw, lane);
#pragma unroll
        for (int m = 0; m < E; ++m) tile[c * tsize + RowLds<real, M>::tile_index(lane + m * L, row, R)] = out[m];
      }
      __syncthreads();
#pragma unroll
      for (int c = 0; c < NOUT; ++c) {
        if (OP == RO_X_IN && c >= X.nout) break;
#pragma unroll
        for (int i = 0; i < E; ++i) {
          const int idx = threadIdx.x + i * blockDim.x;
          const int r = idx & (R - 1), k = idx >> logR;
          stc<real>(spec + (size_t)c * M * ny, (unsigned)(k * ny + y0 + r),
                    tile[c * tsize + RowLds<real, M>::tile_index(k, r, R)]);
        }
      }
    } else {
#pragma unroll
    for (int c = 0; c < NOUT; ++c) {
      if (OP == RO_X_IN && c >= X.nout) break;
      const int tid = opaque(threadIdx.x), lane = tid & (L - 1);
      if constexpr (RowLds<real, M>::ALIAS) __syncthreads();
      reg_fft<real, false, M, E>(v[c], xa, lane, tw, 2);
      C out[E];
      r2c_bins<real, M, E>(v[c], out, tw, lane);
      __syncthreads();  // the tile is free
#pragma unroll
      for (int m = 0; m < E; ++m) tile[RowLds<real, M>::tile_index(lane + m * L, row, R)] = out[m];
      __syncthreads();
      // transposed store: spec[c][kx][y0 + r], r fastest
      for (int idx = tid; idx < M * R; idx += blockDim.x) {
        const int r = idx & (R - 1), k = idx >> logR;
        stc<real>(spec + (size_t)c * M * ny, (unsigned)(k * ny + y0 + r), tile[RowLds<real, M>::tile_index(k, r, R)]);
      }
    }
    }
    block_reduce_store<NP_ROW>(acc, red, part + (size_t)s * NP_ROW * ngr + g, ngr, op_nacc(OP), op_maxslot(OP));
    asm volatile("; end of row op %0" ::"i"(OP));  // keeps the copies apart
  };
#define SPFF_ROW_PASS(OPC) pass(std::integral_constant<int, OPC>{})
  SPFF_ROW_SWITCH(X.op, SPFF_ROW_PASS)
#undef SPFF_ROW_PASS
}

// Algorithmic HBM bytes per pixel moved by the row kernel's forward part,
// the column kernel and the row kernel's inverse part in a tick that
// finishes phase `inv` and starts `phase` (r = sizeof(real)): every input
// plane read once, every output plane written once, half spectra (nx/2 * ny
// complex values = r bytes per pixel per component) written by the forward
// part, read and written by the column kernel, read by the inverse part.
__device__ inline void phase_bytes(int inv, int phase, int flags, int split, double r, double* b) {
  const int op = row_op(inv, phase);
  const double sp = r;  // half spectrum, per pixel per component
  const double strain = split ? 3 : 0;
  const bool first = flags & FL_THETA_FIRST;
  const int nin = op_comps_in(op, inv), nout = op_comps_out(op, phase);
  double planes = 0.0, bytes = 0.0;
  switch (op) {
    case RO_RES:
      planes = 5 + ((flags & FL_FIRST_OF_STEP) ? 1 : 0) + ((flags & FL_THETA_PENDING) ? 6 + (first ? 0 : 3) : 0);
      break;
    case RO_RES_CG: planes = 2 + strain + 3; break;
    case RO_CG_CG: planes = 2 + strain + 3 + (first ? 0 : 3) + 6; break;
    case RO_ASM: planes = 6 + 4 + ((flags & FL_NE_SCALE) ? 3 : 0); break;
    case RO_ASM_PQ: planes = 4 + 1; break;
    case RO_ASM_WAIT: planes = 4 + 2; break;
    case RO_R_PQ:
      planes = 6 + 1;
      bytes = 1;
      break;
    case RO_PQ: planes = 2; break;
    case RO_PFR:
      planes = 3 + ((flags & FL_PF_FIRST) ? 0 : 1) + 2;
      bytes = (flags & FL_PF_FIRST) ? 0 : 1;
      break;
    case RO_AM:
    case RO_RESTORE: planes = 2; break;
    case RO_STATS: planes = 5; break;
    default: break;
  }
  b[0] = planes * r + bytes + nout * sp;
  // column kernel: spectra in, result out; mechanics: the residual's spectrum
  // out, and in after the first
  const bool mech = phase == PH_M_RES || phase == PH_M_CG;
  b[1] = nout * sp * ((phase == PH_PF_PQ || phase == PH_STATS) ? 1.0 : (phase == PH_M_CG ? 4.0 : (mech ? 3.0 : 2.0)));
  b[2] = nin * sp;
}

// ===========================================================================
// Controller of one slot, run by one wavefront.  Reduces the tick's partials
// in a fixed order, updates FP64 scalars and moves the slot's state machine.
// It reads no plane: other groups of its launch may be writing them already.
// ===========================================================================
// FP32 mechanics solves stop at this much of their tolerance (the outer and
// the inner one; the attainable-accuracy floor keeps its value).  The norm of
// the residual, summed in Fourier space, is that of its field to 1e-7, but a
// residual that is updated in Fourier space collects less rounding than one
// updated in real space: on elastic steps of 64^2 to 512^2 it ends 0.1 to 1.4%
// smaller after the same iterations.  Without the margin a solve that lies
// that near its tolerance would end an iteration sooner, with the error of one
// iteration less.
template <typename real>
constexpr double MECH_MARGIN = std::is_same<real, float>::value ? 0.97 : 1.0;

// The controller step of slot s after a tick: one wavefront reads the
// tick's partial sums and the control block C, lane 0 writes the advanced
// block back into C: the phase that the next row kernel finishes (inv) and
// the one that it starts (phase).  `writer`: this wavefront also records the
// step's statistics (byte counters, finished load steps, the queue
// position); the other wavefronts that run the same step on their own copy
// of C (every row work-group of the slot) only advance their copy.
template <typename real>
__device__ __forceinline__ void ctrl_slot(int s, const SlotParam* __restrict__ prms, SlotCtl& C, bool writer,
                                          const double* __restrict__ prow, const double* __restrict__ pcol,
                                          double* __restrict__ prof, SlotSeq* __restrict__ seqs,
                                          StepRec* __restrict__ recs, int nx, int ny, int ngr, int ngc,
                                          const EarlyPartials& early) {
  const double* pr = prow + (size_t)s * NP_ROW * ngr;
  const double* pc = pcol + (size_t)s * NP_COL * ngc;
  const int phase = uni(C.phase), inv = uni(C.inv);
  if (phase == PH_IDLE) return;
  if (threadIdx.x == 0 && C.ticks == 0 && C.t_start == 0) C.t_start = wall_clock64();
  const SlotParam& P = prms[s];
  if (prof && writer && threadIdx.x == 0) {
    double b[3];
    phase_bytes(inv, phase, C.flags, P.contact, double(sizeof(real)), b);
    const double npx = double(nx) * double(ny);
    prof[3 * s + 0] += b[0] * npx;
    prof[3 * s + 1] += b[1] * npx;
    prof[3 * s + 2] += b[2] * npx;
  }
  const double inv_n = 1.0 / (double(nx) * double(ny));
  // the sums of the tick: those of the row kernel's op, and the column
  // kernel's; all lanes compute the same values, lane 0 writes
  double o[NP_ROW], oc;
  {
    const int op = row_op(inv, phase);
    const bool col = phase == PH_M_RES || phase == PH_M_CG || phase == PH_PF_PQ || phase == PH_STATS;
    reduce_partials(pr, ngr, op_nacc(op), op_maxslot(op), pc, col ? ngc : 0, early, o, &oc);
  }
  int nphase = phase, ninv = PH_IDLE;
  int flags = uni(C.flags);
  int cg = C.cg, cg_newton = C.cg_newton, newton = C.newton, bccg = C.bccg, pf_it = C.pf_it, am = C.am;
  int newton_solve = C.newton_solve;
  int status = C.status;
  double mech_ref = C.mech_ref, mech_target = C.mech_target, mech_res = C.mech_res, rr = C.rr;
  double inner_tol = C.inner_tol, alpha_m = C.alpha_m, beta_m = C.beta_m;
  double pf_ref = C.pf_ref, pf_target = C.pf_target, pf_res = C.pf_res, rr_pf = C.rr_pf;
  double alpha_pf = C.alpha_pf, beta_pf = C.beta_pf, pq = C.pq, rp = C.rp, dphi = C.dphi;
  double pf_bnorm = C.pf_bnorm, pf_best = C.pf_best, mech_floor = C.mech_floor, pf_floor = C.pf_floor;
  int pf_best_it = C.pf_best_it;
  double eta_dt = C.eta_dt, dt = C.dt;
  int halvings = C.halvings, advance = C.advance;
  double gamma = C.gamma, fmax_ne = C.fmax_ne, dmax = C.dmax;
  int ne_flag = C.ne_flag;
  bool scaled = false;
  bool bad = false;
  auto pf_done = [&]() {
    if (flags & FL_INIT_SOLVE) {
      flags &= ~FL_INIT_SOLVE;
      nphase = PH_IDLE;
    } else {
      nphase = PH_AM_CHK;
    }
  };
  switch (phase) {
    case PH_M_RES: {
      const double sh2 = o[0], sg2 = o[1], r2 = oc * inv_n;  // Parseval
      bad = !isfinite(sh2) || !isfinite(r2) || !isfinite(sg2);
      mech_res = sqrt(r2);
      // G[sigma] cannot be evaluated more accurately than the rounding of
      // sigma and of the transforms: below that floor the solve is done
      mech_floor = P.floor_coef * sqrt(sg2);
      if (!(flags & FL_MECH_STARTED)) {
        // first residual of this mechanics solve fixes the reference norm
        mech_ref = fmax(sqrt(sh2), mech_res);
        mech_target = MECH_MARGIN<real> * (P.tol_mech * mech_ref + P.tol_abs_mech);
        flags |= FL_MECH_STARTED;
        newton_solve = 0;
      }
      flags &= ~(FL_FIRST_OF_STEP | FL_THETA_PENDING | FL_THETA_FIRST);
      if (mech_res <= fmax(mech_target, mech_floor)) {
        nphase = PH_PF_ASM;
      } else if (newton_solve >= P.max_newton) {
        flags |= FL_NOT_CONVERGED;
        nphase = PH_PF_ASM;
      } else {
        inner_tol = (P.contact == 0) ? fmax(mech_target, mech_floor)
                                   : fmax(0.1 * MECH_MARGIN<real> * mech_res, fmax(mech_target, mech_floor));
        rr = r2;
        cg_newton = 0;
        ninv = PH_M_RES;
        nphase = PH_M_CG;
      }
      if (nphase == PH_PF_ASM) flags &= ~FL_MECH_STARTED;
      break;
    }
    case PH_M_CG: {
      const double pcp = o[0], r2 = oc * inv_n;  // Parseval
      bad = !isfinite(pcp) || !isfinite(r2);
      alpha_m = cg_alpha(pcp, rr);
      ++cg;
      ++cg_newton;
      flags &= ~FL_THETA_FIRST;
      if (cg_newton == 1) flags |= FL_THETA_FIRST;
      beta_m = (rr > 0.0) ? r2 / rr : 0.0;
      rr = r2;
      if (sqrt(r2) <= inner_tol || cg_newton >= P.max_cg || pcp <= 0.0) {
        // the next M_RES applies theta + alpha p
        if (sqrt(r2) > inner_tol) flags |= FL_NOT_CONVERGED;
        ++newton;
        ++newton_solve;
        flags |= FL_THETA_PENDING;
        nphase = PH_M_RES;
      } else {
        ninv = PH_M_CG;
        nphase = PH_M_CG;
      }
      break;
    }
    case PH_PF_ASM: {
      flags &= ~FL_NE_SCALE;
      bad = !isfinite(o[0]);
      pf_bnorm = sqrt(o[0]);
      dmax = o[1];
      ninv = PH_PF_ASM;
      if (flags & FL_NE_CHECK) {
        nphase = PH_PF_WAIT;
      } else {
        // the first direction is -r: start the first iteration with it
        flags |= FL_PF_FIRST;
        nphase = PH_PF_PQ;
      }
      break;
    }
    case PH_PF_WAIT:
    case PH_PF_PQ: {
      const double r2 = o[0];
      if (phase == PH_PF_WAIT) {
        // Algorithm 4: -F_phi(phi_n, eps_n) and the crack driving force
        // -h'(phi_n) psi0+ were evaluated by this assembly
        flags &= ~FL_NE_CHECK;
        fmax_ne = o[1];
        if (fmax_ne > P.fphi_max && dmax > P.drive_thr) ne_flag = 1;
        // the factor that the column kernel left (col_ne_gamma), below 0: none
        if (fmax_ne > P.fphi_max && ne_flag && pc[0] >= 0.0) {
          gamma = pc[0];
          scaled = true;
          flags |= FL_NE_SCALE;
          nphase = PH_PF_ASM;  // assemble again at the scaled strain
          break;
        }
      }
      if (inv != PH_IDLE) {
        // the residual that this tick's row kernel finished
        bad = !isfinite(r2);
        rr_pf = r2;
        pf_res = sqrt(r2);
        // attainable accuracy of r = J phi - b in the working precision
        pf_floor = P.floor_coef * (sqrt(o[3]) + P.kappa * P.lap_rms * sqrt(o[2]) + pf_bnorm);
        bool done = false;
        if (inv == PH_PF_ASM) {
          pf_ref = fmax(pf_bnorm, pf_res);
          pf_target = P.tol_pf * pf_ref + P.tol_abs_pf;
          pf_it = 0;
          pf_best = pf_res;
          pf_best_it = 0;
          done = pf_res <= fmax(pf_target, pf_floor);
        } else {
          bad |= !isfinite(o[1]);
          beta_pf = bccg_beta(r2, o[1], C);
          ++pf_it;
          ++bccg;
          if (pf_res < pf_best) {
            pf_best = pf_res;
            pf_best_it = pf_it;
          }
          if (pf_res <= fmax(pf_target, pf_floor)) {
            done = true;
          } else if (P.stall_iters > 0 && pf_it - pf_best_it >= P.stall_iters) {
            flags |= FL_STALLED;
            done = true;
          } else if (pf_it >= P.max_bccg) {
            flags |= FL_NOT_CONVERGED;
            done = true;
          }
        }
        if (done) {
          flags &= ~FL_PF_FIRST;
          pf_done();
          break;
        }
        if (phase == PH_PF_WAIT) {
          flags |= FL_PF_FIRST;
          nphase = PH_PF_PQ;
          break;
        }
      }
      // p = -r + beta m p_old: sum d p^2 and r.p from the sums over r and
      // m p_old, sum L |p^|^2 from the column kernel
      const double b = (flags & FL_PF_FIRST) ? 0.0 : beta_pf;
      const double dpp = o[4] - 2.0 * b * o[5] + b * b * o[6];
      rp = -r2 + b * o[7];
      bad |= !isfinite(dpp) || !isfinite(rp) || !isfinite(oc);
      pq = dpp + P.kappa * inv_n * oc;
      if (!(pq > 0.0)) {
        flags |= FL_NOT_CONVERGED;
        flags &= ~FL_PF_FIRST;
        pf_done();
      } else {
        alpha_pf = -rp / pq;
        nphase = PH_PF_R;
      }
      break;
    }
    case PH_PF_R:
      flags &= ~FL_PF_FIRST;
      ninv = PH_PF_R;
      nphase = PH_PF_PQ;
      break;
    case PH_AM_CHK: {
      dphi = o[0];
      bad = !isfinite(dphi);
      ++am;
      if (P.evolution == 2) {
        advance = dphi < P.dphi_min ? 1 : 0;
        nphase = PH_STATS;
        break;
      }
      if (P.evolution == 1) {
        // Algorithm 3: accept the phase field if its change is small enough
        // or dt has reached its floor, else retry from phi_n with dt / 2
        if (dphi < P.dphi_max || dt <= P.dt_min) {
          if (dphi < 0.5 * P.dphi_max) dt = fmin(2.0 * dt, P.dt_max);
          advance = (dphi < P.dphi_min && dt >= P.dt_max) ? 1 : 0;
          nphase = PH_STATS;
        } else {
          dt *= 0.5;
          ++halvings;
          eta_dt = P.eta / dt;
          nphase = PH_TD_RESTORE;
        }
        break;
      }
      if (dphi <= P.tol_am) {
        nphase = PH_STATS;
      } else if (am >= P.max_am) {
        flags |= FL_NOT_CONVERGED;
        nphase = PH_STATS;
      } else {
        nphase = PH_M_RES;
      }
      break;
    }
    case PH_TD_RESTORE:
      nphase = PH_PF_ASM;
      break;
    case PH_X_PROJ:
    case PH_X_DISP:
    case PH_X_LAP:
      ninv = phase;
      nphase = PH_X_END;
      break;
    case PH_X_END:
      nphase = PH_IDLE;
      break;
    case PH_STATS: {
      bad = false;
      for (int i = 0; i < 8; ++i) bad |= !isfinite(o[i]);
      if (threadIdx.x == 0) {
        C.F_e = o[0];
        C.F_f = P.cwl * (o[1] + P.ell * P.ell * inv_n * oc);
        C.phi_sum = o[2];
        C.phi_max = o[3];
        C.crack_px = o[4];
        C.sbar[0] = o[5] * inv_n;
        C.sbar[1] = o[6] * inv_n;
        C.sbar[2] = o[7] * inv_n;
      }
      nphase = PH_IDLE;
      break;
    }
    default:
      break;
  }
  if (bad) {
    flags |= FL_NONFINITE;
    status = -4;
    nphase = PH_IDLE;
  }
  uint64_t t_end = C.t_end;
  if (nphase == PH_IDLE) {
    ninv = PH_IDLE;
    t_end = wall_clock64();
  }
  // a load step just ended: record it and start the next one of the queue
  bool restart = false;
  if (seqs && nphase == PH_IDLE && (phase == PH_STATS || bad) && !(flags & FL_INIT_SOLVE) && threadIdx.x == 0 &&
      C.seq_pos < seqs[s].len) {
    const int pos = C.seq_pos;
    if (writer) {
      StepRec& r = recs[(size_t)s * SEQ_MAX + pos];
      r.status = status;
      r.flags = flags;
      r.am = am;
      r.newton = newton;
      r.cg = cg;
      r.bccg = bccg;
      r.ticks = C.ticks + 1;
      r.dt = dt;
      r.halvings = halvings;
      r.advance = advance;
      r.gamma = gamma;
      r.fmax_ne = fmax_ne;
      r.ne_flag = ne_flag;
      r.t_start = C.t_start;
      r.t_end = t_end;
      r.dphi = dphi;
      r.mech_res = mech_res;
      r.pf_res = pf_res;
      r.F_e = C.F_e;
      r.F_f = C.F_f;
      for (int k = 0; k < 3; ++k) {
        r.sbar[k] = C.sbar[k];
        r.eps_bar[k] = C.eps_bar[k];
      }
      r.phi_sum = C.phi_sum;
      r.phi_max = C.phi_max;
      r.crack_px = C.crack_px;
      seqs[s].pos = pos + 1;
    }
    C.seq_pos = pos + 1;
    if (pos + 1 < seqs[s].len && status >= 0) restart = true;
  }
  if (restart) {
    // fresh control block for the next load step of the queue
    const SlotSeq& q = seqs[s];
    const int pos = C.seq_pos;
    if (q.incr) {
      // evolution queue: the next step continues from this step's final
      // macroscopic strain, plus the increment if the algorithm advances
      const double a = advance ? 1.0 : 0.0;
      C.eps_bar[0] += a * q.eps_bar[pos][0];
      C.eps_bar[1] += a * q.eps_bar[pos][1];
      C.eps_bar[2] += a * q.eps_bar[pos][2];
    } else {
      C.eps_bar[0] = q.eps_bar[pos][0];
      C.eps_bar[1] = q.eps_bar[pos][1];
      C.eps_bar[2] = q.eps_bar[pos][2];
    }
    C.phase = PH_M_RES;
    C.inv = PH_IDLE;
    C.flags = FL_FIRST_OF_STEP | (P.evolution == 2 ? FL_NE_CHECK : 0);
    C.am = C.newton = C.cg = C.bccg = C.cg_newton = C.pf_it = C.newton_solve = 0;
    C.ticks = 0;
    C.status = 0;
    C.dphi = 0.0;
    C.dt = dt;
    C.halvings = 0;
    C.advance = 0;
    C.eta_dt = P.evolution == 1 ? P.eta / dt : (P.evolution == 2 ? P.eta / P.dt_max : P.eta_dt);
    C.gamma = 1.0;
    C.fmax_ne = 0.0;
    C.ne_flag = ne_flag;
    C.t_start = wall_clock64();
    return;
  }
  if (threadIdx.x == 0) {
    C.phase = nphase;
    C.inv = ninv;
    C.flags = flags;
    C.cg = cg;
    C.cg_newton = cg_newton;
    C.newton = newton;
    C.bccg = bccg;
    C.pf_it = pf_it;
    C.newton_solve = newton_solve;
    C.am = am;
    C.status = status;
    C.mech_ref = mech_ref;
    C.mech_target = mech_target;
    C.mech_res = mech_res;
    C.rr = rr;
    C.inner_tol = inner_tol;
    C.alpha_m = alpha_m;
    C.beta_m = beta_m;
    C.pf_ref = pf_ref;
    C.pf_target = pf_target;
    C.pf_res = pf_res;
    C.rr_pf = rr_pf;
    C.alpha_pf = alpha_pf;
    C.beta_pf = beta_pf;
    C.pq = pq;
    C.rp = rp;
    C.dphi = dphi;
    C.pf_bnorm = pf_bnorm;
    C.pf_best = pf_best;
    C.pf_best_it = pf_best_it;
    C.mech_floor = mech_floor;
    C.pf_floor = pf_floor;
    C.eta_dt = eta_dt;
    C.dt = dt;
    C.halvings = halvings;
    C.advance = advance;
    C.gamma = gamma;
    C.fmax_ne = fmax_ne;
    C.dmax = dmax;
    C.ne_flag = ne_flag;
    if (scaled) {
      C.eps_bar[0] *= gamma;
      C.eps_bar[1] *= gamma;
      C.eps_bar[2] *= gamma;
    }
    C.ticks = C.ticks + 1;
    C.t_end = t_end;
  }
}

// ===========================================================================
// Kernel entry points: the bodies above, stamped with the device clock when
// profiling (kt != nullptr).
// ===========================================================================
__device__ __forceinline__ int kt_line() {
  return (blockIdx.x + blockIdx.y * 29) & (KT_LINES - 1);
}
__device__ __forceinline__ void kt_begin(KTime* kt) {
  if (kt && threadIdx.x == 0)
    atomicMin(&kt->start[kt_line() * KT_STRIDE], (unsigned long long)wall_clock64());
}
__device__ __forceinline__ void kt_end(KTime* kt) {
  if (kt) {
    __syncthreads();
    if (threadIdx.x == 0) atomicMax(&kt->end[kt_line() * KT_STRIDE], (unsigned long long)wall_clock64());
  }
}

// Folds the times of one tick (kt[0..2]: row-forward part, column kernel,
// row-inverse part) into ktsum and resets the words for the tick after next;
// one wavefront, lane l takes line l.  ktsum[j]: activity of part j (first
// start to last end); ktsum[4 + j]: its span (first start to the first start
// of the part after it; t_next for the column kernel).
__device__ __forceinline__ void kt_fold(KTime* kt, unsigned long long t_next, unsigned long long* ktsum) {
  const int l = threadIdx.x & 63;
  unsigned long long st[3], en[3];
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    unsigned long long a = kt[j].start[l * KT_STRIDE], b = kt[j].end[l * KT_STRIDE];
    kt[j].start[l * KT_STRIDE] = ~0ull;
    kt[j].end[l * KT_STRIDE] = 0ull;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
      const unsigned long long a2 = __shfl_xor(a, off, 64), b2 = __shfl_xor(b, off, 64);
      a = a2 < a ? a2 : a;
      b = b2 > b ? b2 : b;
    }
    st[j] = a;
    en[j] = b;
  }
  if (l == 0) {
    const unsigned long long nxt[3] = {st[1], t_next, st[0]};
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      if (en[j] > st[j]) ktsum[j] += en[j] - st[j];
      if (nxt[j] > st[j] && nxt[j] != ~0ull) ktsum[4 + j] += nxt[j] - st[j];
    }
  }
}
// First start stamped in kt (one wavefront).
__device__ __forceinline__ unsigned long long kt_first_start(const KTime* kt) {
  unsigned long long a = kt->start[(threadIdx.x & 63) * KT_STRIDE];
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    const unsigned long long a2 = __shfl_xor(a, off, 64);
    a = a2 < a ? a2 : a;
  }
  return a;
}

// Timer bookkeeping of the column kernel: with timers on, the launch has one
// extra row of work-groups; its group 0 folds the previous tick's times
// (kt_prev, null for the first tick of a block) -- the previous tick ended
// before this tick's row kernel, whose first start (kt_row) closes the
// previous column kernel's span -- and the other extra groups return.
struct ColTimers {
  KTime* kt;             // this column kernel's stamps
  KTime* kt_prev;        // the previous tick's three parts
  const KTime* kt_row;   // this tick's row kernel (its inverse part starts it)
  unsigned long long* ktsum;
};
__device__ __forceinline__ bool col_timer_group(const ColTimers& T) {
  if (!T.kt || blockIdx.y != gridDim.y - 1) return false;
  if (T.kt_prev && blockIdx.x == 0 && threadIdx.x < 64) kt_fold(T.kt_prev, kt_first_start(T.kt_row), T.ktsum);
  return true;
}

// Between the parts of a row kernel (every thread of a group that has work).
__device__ __forceinline__ void row_middle(const RowTimers& T) {
  if (T.inv) {
    kt_end(T.inv);
    kt_begin(T.fwd);
  }
}

template <typename real>
__global__ __launch_bounds__(THREADS) void k_row(const int* __restrict__ list, const SlotPtr<real>* __restrict__ ptrs,
                                                 const SlotParam* __restrict__ prms, const CtrlArgs A,
                                                 const cplx<real>* __restrict__ twx, double* __restrict__ part,
                                                 int nx, int ny, int R, int ngr, const RowTimers T) {
  kt_begin(T.inv);
  k_row_body<real>(list, ptrs, prms, A, twx, part, nx, ny, R, ngr, T);
  kt_end(T.fwd);
}

// Wavefronts per SIMD that the register rows are compiled for.  Eight FP32
// points per lane want 131 to 134 registers; held to 128 (15 of them kept in
// scratch memory at 256 points) a CU takes four work-groups instead of three:
// 64 x 512^2 119 us a tick's part against 125.  512 points would not gain a
// group (LDS), and 16 points per lane lose 2% at three wavefronts.
template <typename real, int M, int E>
constexpr int ROW_WAVES = std::is_same<real, float>::value && E == 8 && M <= 256 ? 4 : 1;
template <typename real, int M, int E>
__global__ __launch_bounds__(THREADS, (ROW_WAVES<real, M, E>)) void k_rowr(const int* __restrict__ list, const SlotPtr<real>* __restrict__ ptrs,
                                                  const SlotParam* __restrict__ prms, const CtrlArgs A,
                                                  const cplx<real>* __restrict__ twx, double* __restrict__ part,
                                                  int ny, int ngr, const RowTimers T) {
  kt_begin(T.inv);
  k_rowr_body<real, M, E>(list, ptrs, prms, A, twx, part, ny, ngr, T);
  kt_end(T.fwd);
}

template <typename real>
__global__ __launch_bounds__(THREADS) void k_col(const int* __restrict__ list, const SlotPtr<real>* __restrict__ ptrs,
                                                 const SlotParam* __restrict__ prms,
                                                 const SlotCtl* __restrict__ ctls,
                                                 const cplx<real>* __restrict__ twy,
                                                 const double* __restrict__ part_row, double* __restrict__ part,
                                                 int nx, int ny, int W, int ngr, int ngc, int nyq_free,
                                                 const ColTimers T) {
  if (col_timer_group(T)) return;
  kt_begin(T.kt);
  k_col_body<real>(list, ptrs, prms, ctls, twy, part_row, part, nx, ny, W, ngr, ngc, nyq_free);
  kt_end(T.kt);
}

template <typename real, int N, int E, bool AHEAD>
__global__ __launch_bounds__(THREADS) void k_colr(const int* __restrict__ list, const SlotPtr<real>* __restrict__ ptrs,
                                                  const SlotParam* __restrict__ prms,
                                                  const SlotCtl* __restrict__ ctls,
                                                  const cplx<real>* __restrict__ twy,
                                                  const double* __restrict__ part_row, double* __restrict__ part,
                                                  int nx, int ngr, int ngc, int nyq_free, const ColTimers T) {
  if (col_timer_group(T)) return;
  kt_begin(T.kt);
  k_colr_body<real, N, E, AHEAD>(list, ptrs, prms, ctls, twy, part_row, part, nx, ngr, ngc, nyq_free);
  kt_end(T.kt);
}

// Closing kernel of a run of ticks: the controller step of the last tick,
// one work-group per listed slot (list null: every slot), from A.ctl_in into
// A.ctl_out (buffer 0, possibly the same block) and the host's mirror.  With timers on, the second wavefront of group 0 folds
// the last tick's kernel times meanwhile.
template <typename real>
__global__ __launch_bounds__(128) void k_close(const int* __restrict__ list, const SlotParam* __restrict__ prms,
                                              const CtrlArgs A, int nx, int ny, int ngr, KTime* kt_last,
                                              unsigned long long* __restrict__ ktsum) {
  constexpr int NW = (int)(sizeof(SlotCtl) / sizeof(int));
  __shared__ SlotCtl lc;
  const unsigned long long t_close = wall_clock64();
  const int s = list ? list[blockIdx.x] : (int)blockIdx.x;
  int* w = reinterpret_cast<int*>(&lc);
  if (s >= 0) {
    const int* src = reinterpret_cast<const int*>(A.ctl_in + s);
    for (int i = threadIdx.x; i < NW; i += blockDim.x) w[i] = src[i];
  }
  __syncthreads();
  if (threadIdx.x < 64) {
    if (s >= 0) {
      if (lc.pending) {
        EarlyPartials early;
        early.load(A.prow + (size_t)s * NP_ROW * ngr, ngr, A.pcol + (size_t)s * NP_COL * A.ngc, A.ngc);
        ctrl_slot<real>(s, prms, lc, true, A.prow, A.pcol, A.prof, A.seqs, A.recs, nx, ny, ngr, A.ngc, early);
      }
      if (threadIdx.x == 0) lc.pending = 0;
    }
  } else if (kt_last && blockIdx.x == 0) {
    kt_fold(kt_last, t_close, ktsum);
  }
  __syncthreads();
  if (s >= 0) {
    int* out = reinterpret_cast<int*>(A.ctl_out + s);
    int* host = A.mirror ? reinterpret_cast<int*>(A.mirror + s) : nullptr;
    for (int i = threadIdx.x; i < NW; i += blockDim.x) {
      out[i] = w[i];
      if (host) host[i] = w[i];
    }
  }
}

// ===========================================================================
// Small utility kernels
// ===========================================================================
// Count non-finite or non-positive entries (E validation).
template <typename real>
__global__ void k_validate(const real* __restrict__ a, size_t n, real lo_excl, real lo_incl, real hi_incl,
                           unsigned int* __restrict__ bad) {
  unsigned int cnt = 0;
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
    const real v = a[i];
    const bool ok = isfinite(v) && v > lo_excl && v >= lo_incl && v <= hi_incl;
    cnt += ok ? 0u : 1u;
  }
  if (cnt) atomicAdd(bad, cnt);
}

// Whole-handle moves between the slots' planes and the caller's buffers: one
// launch for all slots (blockIdx.y).  A copy and a kernel per slot and plane
// cost 8 us of gap each: 1.9 ms to restore and 1.3 ms to read out the state
// of 64 problems of 512^2 that move in 0.2 ms.  VEC values per access: 16
// bytes where every caller buffer is aligned to them, else one.
template <typename real, int VEC>
struct VecOf {
  typedef real type __attribute__((ext_vector_type(VEC)));
};
template <typename real>
struct VecOf<real, 1> {
  typedef real type;
};

// Slot planes of the resident state.
template <typename real>
struct StatePlanes {
  unsigned char* base;  // slot 0
  size_t slot_bytes;
  size_t eps, phi, phi_ref;  // byte offsets in a slot
  __device__ __forceinline__ real* plane(int s, int k, int n) const {
    unsigned char* b = base + (size_t)s * slot_bytes;
    return k < 3 ? reinterpret_cast<real*>(b + eps) + (size_t)k * n
                 : reinterpret_cast<real*>(b + (k == 3 ? phi : phi_ref));
  }
};

// Values that the library takes as input: finite, and in FP64 at most 1e300
// in size (any finite FP32 value: 1e300 rounds to infinity there).
template <typename real>
__device__ __forceinline__ bool acceptable(real v) {
  return isfinite(v) && fabs(v) <= real(1e300);
}

// *flag = token if a value is not acceptable.
template <typename real>
__global__ void k_check_finite(const real* __restrict__ a, size_t n, unsigned* __restrict__ flag, unsigned token) {
  bool bad = false;
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
    bad |= !acceptable(a[i]);
  if (bad) *flag = token;
}

// State (eps*[3], phi, phi_ref per slot) in (PUT; not if *flag is token) or
// out; *refused tells the host which.
template <typename real, int VEC, bool PUT>
__global__ void k_state(const StatePlanes<real> P, real* __restrict__ ext, int n, const unsigned* __restrict__ flag,
                        unsigned token, unsigned* __restrict__ refused) {
  using V = typename VecOf<real, VEC>::type;
  const int s = blockIdx.y;
  if constexpr (PUT) {
    const bool no = *flag == token;
    if (blockIdx.x == 0 && s == 0 && threadIdx.x == 0) *refused = no ? 1u : 0u;
    if (no) return;
  }
  for (int k = 0; k < 5; ++k) {
    V* in = reinterpret_cast<V*>(P.plane(s, k, n));
    V* out = reinterpret_cast<V*>(ext + ((size_t)s * 5 + k) * n);
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n / VEC; i += gridDim.x * blockDim.x) {
      if constexpr (PUT)
        in[i] = out[i];
      else
        out[i] = in[i];
    }
  }
}

// Output fields (see SPFF_FIELD_*) of slots s0 + blockIdx.y; out[f] null: not
// asked for.
template <typename real, int VEC>
__global__ void k_fields(const SlotPtr<real>* __restrict__ ptrs, const SlotParam* __restrict__ prms,
                         const SlotCtl* __restrict__ ctls, int s0, int n, const FieldOut<real> O) {
  using V = typename VecOf<real, VEC>::type;
  const int slot = s0 + blockIdx.y;
  const SlotPtr<real> F = ptrs[slot];
  const SlotParam& P = prms[slot];
  const SlotCtl& C = ctls[slot];
  const real lt = real(P.lam_t), mt = real(P.mu_t), kres = real(P.k_res);
  const size_t j = blockIdx.y;
  auto ld = [](const real* p, int i, real* x) {
    V v = reinterpret_cast<const V*>(p)[i];
    __builtin_memcpy(x, &v, sizeof(v));
  };
  auto st = [](real* p, int i, const real* x) {
    V v;
    __builtin_memcpy(&v, x, sizeof(v));
    reinterpret_cast<V*>(p)[i] = v;
  };
  const bool law = O.strain || O.stress || O.psi, need_eps = law || O.eps, need_phi = O.phi || O.stress;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n / VEC; i += gridDim.x * blockDim.x) {
    real ph[VEC], x[3][VEC];
    if (need_phi) ld(F.phi, i, ph);
    if (O.phi) st(O.phi + j * n, i, ph);
    if (O.phi_ref) {
      real r[VEC];
      ld(F.phi_ref, i, r);
      st(O.phi_ref + j * n, i, r);
    }
    if (!need_eps) continue;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      ld(F.eps + (size_t)k * n, i, x[k]);
      if (O.eps) st(O.eps + (j * 3 + k) * n, i, x[k]);
    }
    if (!law) continue;
    real E[VEC], psi[VEC], sg[3][VEC];
    if (O.stress || O.psi) ld(F.E, i, E);
#pragma unroll
    for (int v = 0; v < VEC; ++v) {
#pragma unroll
      for (int k = 0; k < 3; ++k) x[k][v] = real(C.eps_bar[k]) + x[k][v];
      const Sym<real> e = {x[0][v], x[1][v], x[2][v]};
      if (O.stress || O.psi) {
        const real lam = lt * E[v], mu = mt * E[v];
        if (O.stress) {
          const real hk = (real(1) - ph[v]) * (real(1) - ph[v]) + kres;
          const Sym<real> t = stress(e, lam, mu, hk, P.contact);
          sg[0][v] = t.xx;
          sg[1][v] = t.yy;
          sg[2][v] = t.xy;
        }
        if (O.psi) {
          real pm;
          energies(e, lam, mu, P.split, &psi[v], &pm);
        }
      }
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      if (O.strain) st(O.strain + (j * 3 + k) * n, i, x[k]);
      if (O.stress) st(O.stress + (j * 3 + k) * n, i, sg[k]);
    }
    if (O.psi) st(O.psi + j * n, i, psi);
  }
}

// Fills nplanes planes of each slot: plane 0 from E (zero without), planes 1
// and 2 from phi (zero without), the rest with zeros; counts the values of E
// that are not positive and acceptable in bad[0], those of phi outside [0, 1]
// in bad[1].
template <typename real>
__global__ void k_init(unsigned char* __restrict__ base, size_t slot_bytes, const real* __restrict__ E,
                       const real* __restrict__ phi, int n, int nplanes, unsigned* __restrict__ bad) {
  const int s = blockIdx.y;
  real* dst = reinterpret_cast<real*>(base + (size_t)s * slot_bytes);
  unsigned bad_e = 0, bad_p = 0;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
    real e = 0, f = 0;
    if (E) {
      e = E[(size_t)s * n + i];
      bad_e += (acceptable(e) && e > real(0)) ? 0u : 1u;
    }
    if (phi) {
      f = phi[(size_t)s * n + i];
      bad_p += (isfinite(f) && f >= real(0) && f <= real(1)) ? 0u : 1u;
    }
    dst[i] = e;
    for (int k = 1; k < nplanes; ++k) dst[(size_t)k * n + i] = k < 3 ? f : real(0);
  }
  if (bad_e) atomicAdd(bad, bad_e);
  if (bad_p) atomicAdd(bad + 1, bad_p);
}

// Words from pinned host memory to the device: a small upload without the
// gaps of a copy command (8 to 12 us on either side).
__global__ void k_upload(const int* __restrict__ src, int* __restrict__ dst, int n) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) dst[i] = src[i];
}

// Sets up a diagnostic operator (phase) over `count` slots from s0, padded
// to `listed` list entries: list, control blocks and pointer table of its
// own, with the caller's buffers as the planes it reads (theta) and writes
// (rm).
template <typename real>
__global__ void k_op_setup(int* __restrict__ list, SlotCtl* __restrict__ ctl, SlotPtr<real>* __restrict__ optr,
                           const SlotPtr<real>* __restrict__ ptrs, int s0, int count, int listed, int phase,
                           const real* __restrict__ in, size_t in_stride, real* __restrict__ out, size_t out_stride) {
  const int j = blockIdx.x;
  if (j >= count) {
    if (threadIdx.x == 0) list[j] = -1;
    return;
  }
  int* c = reinterpret_cast<int*>(ctl + s0 + j);
  for (int i = threadIdx.x; i < (int)(sizeof(SlotCtl) / sizeof(int)); i += blockDim.x) c[i] = 0;
  __syncthreads();
  if (threadIdx.x == 0) {
    list[j] = s0 + j;
    ctl[s0 + j].phase = phase;
    SlotPtr<real> F = ptrs[s0 + j];
    if (in) F.theta = const_cast<real*>(in) + j * in_stride;
    if (out) F.rm = out + j * out_stride;
    optr[s0 + j] = F;
  }
}

// ===========================================================================
// Host-side launchers (called from the C-ABI implementation).
// ===========================================================================

template <typename real>
hipError_t launch_tick(const LaunchGeom& G, const TickBufs<real>& B, int i, hipStream_t st, int kernels) {
  // tick i reads control block (i & 1) and the partials of tick i - 1
  // (row partials double-buffered: this tick's row kernel writes the other
  // half while its groups reduce the previous one)
  const int cur = i & 1, nxt = cur ^ 1;
  CtrlArgs A;
  A.ctl_in = B.ctl[cur];
  A.ctl_out = B.ctl[nxt];
  A.prow = B.prow[nxt];
  A.pcol = B.pcol;
  A.prof = B.prof;
  A.seqs = B.seqs;
  A.recs = B.recs;
  A.post = B.post;
  A.mirror = nullptr;
  A.ngc = G.ngc;
  const int* list = B.list;
  const SlotPtr<real>* ptrs = B.ptrs;
  const SlotParam* prms = B.prms;
  const SlotCtl* ctls = B.ctl[nxt];
  const auto* twx = B.twx;
  const auto* twy = B.twy;
  double* prow = B.prow[cur];
  double* pcol = B.pcol;
  KTime* ktset = B.kt ? B.kt + 3 * cur : nullptr;
  RowTimers TR;
  TR.fwd = ktset;
  TR.inv = ktset ? ktset + 2 : nullptr;
  ColTimers T;
  T.kt = ktset ? ktset + 1 : nullptr;
  T.kt_prev = (B.kt && i > 0) ? B.kt + 3 * nxt : nullptr;
  T.kt_row = TR.inv;
  T.ktsum = B.ktsum;
  dim3 grow(G.ngr, G.S), gcol(G.ngc, G.S + (B.kt ? 1 : 0));
#define SPFF_ROWS(MM, EE)                                                                                    \
  hipLaunchKernelGGL((k_rowr<real, MM, EE>), grow, dim3(G.threads), G.lds_row, st, list, ptrs, prms, A, twx, \
                     prow, G.ny, G.ngr, TR)
  if (!(kernels & TICK_ROW)) {
  } else if (G.row_reg == 2) {
    switch (G.nx) {
      case 128: SPFF_ROWS(64, 4); break;
      case 256: SPFF_ROWS(128, 4); break;
      case 512: SPFF_ROWS(256, 4); break;
      default: return hipErrorInvalidValue;
    }
  } else if (G.row_reg == 1) {
    switch (G.nx) {
      case 128: SPFF_ROWS(64, 8); break;
      case 256: SPFF_ROWS(128, 8); break;
      case 512: SPFF_ROWS(256, 8); break;
      case 1024: SPFF_ROWS(512, 8); break;
      default:
        // FP64 has no register kernel for 2048-point rows
        if constexpr (std::is_same<real, float>::value)
          SPFF_ROWS(1024, 16);
        else
          return hipErrorInvalidValue;
        break;
    }
  } else {
    hipLaunchKernelGGL(k_row<real>, grow, dim3(G.threads), G.lds_row, st, list, ptrs, prms, A, twx, prow, G.nx, G.ny,
                       G.R, G.ngr, TR);
  }
#undef SPFF_ROWS
  if (!(kernels & TICK_COL)) return hipGetLastError();
#define SPFF_COLS(NN, EE, AA)                                                                                           \
  hipLaunchKernelGGL((k_colr<real, NN, EE, AA>), gcol, dim3(G.threads_col), G.lds_col, st, list, ptrs, prms, ctls, twy, \
                     prow, pcol, G.nx, G.ngr, G.ngc, G.nyq_free, T)
#define SPFF_COLS8(NN)        \
  if (ahead)                  \
    SPFF_COLS(NN, 8, true);   \
  else                        \
    SPFF_COLS(NN, 8, false);
  // at most one wavefront per SIMD (FP32: two): registers for loads ahead
  // cost nothing
  const long col_waves = (long)G.ngc * G.S * (G.threads_col / 64);
  const bool ahead = col_waves <= (sizeof(real) == 8 ? 1024 : 2048);
  if (G.col_reg && G.col_pts == 8) {
    switch (G.ny) {
      case 128: SPFF_COLS8(128) break;
      case 256: SPFF_COLS8(256) break;
      case 512: SPFF_COLS8(512) break;
      case 1024: SPFF_COLS8(1024) break;
      default: SPFF_COLS8(2048) break;
    }
  } else if (G.col_reg) {
    // 16 points per lane: plans of FP32 problems only
    if constexpr (std::is_same<real, float>::value) {
      if (G.ny == 1024)
        SPFF_COLS(1024, 16, false);
      else
        SPFF_COLS(2048, 16, false);
    } else {
      return hipErrorInvalidValue;
    }
  } else {
    hipLaunchKernelGGL(k_col<real>, gcol, dim3(G.threads_col), G.lds_col, st, list, ptrs, prms, ctls, twy, prow, pcol,
                       G.nx, G.ny, G.W, G.ngr, G.ngc, G.nyq_free, T);
  }
#undef SPFF_COLS8
#undef SPFF_COLS
  return hipGetLastError();
}

template <typename real>
hipError_t launch_close(const LaunchGeom& G, const TickBufs<real>& B, int k, hipStream_t st, int slots) {
  // after ticks 0..k-1 the latest control blocks are in buffer (k & 1)
  const int last = (k - 1) & 1;
  CtrlArgs A;
  A.ctl_in = B.ctl[k & 1];
  A.ctl_out = B.ctl[0];
  A.prow = B.prow[last];
  A.pcol = B.pcol;
  A.prof = B.prof;
  A.seqs = B.seqs;
  A.recs = B.recs;
  A.post = nullptr;
  A.mirror = B.mirror;
  A.ngc = G.ngc;
  hipLaunchKernelGGL(k_close<real>, dim3(slots > 0 ? slots : G.S), dim3(128), 0, st, slots > 0 ? nullptr : B.list,
                     B.prms, A, G.nx, G.ny, G.ngr, B.kt ? B.kt + 3 * last : nullptr, B.ktsum);
  return hipGetLastError();
}

template <typename real>
hipError_t launch_validate(const real* a, size_t n, double lo_excl, double lo_incl, double hi_incl,
                           unsigned int* bad, hipStream_t st) {
  int blocks = (int)((n + 255) / 256);
  if (blocks > 4096) blocks = 4096;
  if (blocks < 1) blocks = 1;
  hipLaunchKernelGGL(k_validate<real>, dim3(blocks), dim3(256), 0, st, a, n, real(lo_excl), real(lo_incl),
                     real(hi_incl), bad);
  return hipGetLastError();
}

namespace {
// blocks of 256 threads over `count` items per slot, about 4096 in all
dim3 slot_grid(size_t count, int slots) {
  size_t bx = (count + 255) / 256;
  const size_t most = std::max<size_t>(8, 4096 / (size_t)slots);
  return dim3((unsigned)std::min(bx, most), (unsigned)slots);
}
template <typename real>
constexpr int VEC16 = 16 / (int)sizeof(real);
bool aligned16(const void* p) { return reinterpret_cast<uintptr_t>(p) % 16 == 0; }
}  // namespace

template <typename real>
hipError_t launch_fields(const SlotPtr<real>* ptrs, const SlotParam* prms, const SlotCtl* ctls, int s0, int slots,
                         int n, const FieldOut<real>& O, hipStream_t st) {
  const bool wide = aligned16(O.phi) && aligned16(O.phi_ref) && aligned16(O.strain) && aligned16(O.stress) &&
                    aligned16(O.psi) && aligned16(O.eps);
  if (wide)
    hipLaunchKernelGGL((k_fields<real, VEC16<real>>), slot_grid(n / VEC16<real>, slots), dim3(256), 0, st, ptrs, prms,
                       ctls, s0, n, O);
  else
    hipLaunchKernelGGL((k_fields<real, 1>), slot_grid(n, slots), dim3(256), 0, st, ptrs, prms, ctls, s0, n, O);
  return hipGetLastError();
}

template <typename real>
hipError_t launch_state(unsigned char* base, size_t slot_bytes, size_t eps, size_t phi, size_t phi_ref, int slots,
                        int n, const void* in, void* out, unsigned* flag, unsigned token, unsigned* refused,
                        hipStream_t st) {
  const StatePlanes<real> P = {base, slot_bytes, eps, phi, phi_ref};
  constexpr int V = VEC16<real>;
  if (in) {
    const real* a = static_cast<const real*>(in);
    real* ext = const_cast<real*>(a);  // only read
    const size_t cnt = (size_t)slots * 5 * n;
    const size_t blocks = std::min<size_t>((cnt + 255) / 256, 4096);
    hipLaunchKernelGGL(k_check_finite<real>, dim3((unsigned)blocks), dim3(256), 0, st, a, cnt, flag, token);
    if (aligned16(in))
      hipLaunchKernelGGL((k_state<real, V, true>), slot_grid(n / V, slots), dim3(256), 0, st, P, ext, n, flag, token,
                         refused);
    else
      hipLaunchKernelGGL((k_state<real, 1, true>), slot_grid(n, slots), dim3(256), 0, st, P, ext, n, flag, token,
                         refused);
  } else {
    real* ext = static_cast<real*>(out);
    if (aligned16(out))
      hipLaunchKernelGGL((k_state<real, V, false>), slot_grid(n / V, slots), dim3(256), 0, st, P, ext, n, flag, token,
                         refused);
    else
      hipLaunchKernelGGL((k_state<real, 1, false>), slot_grid(n, slots), dim3(256), 0, st, P, ext, n, flag, token,
                         refused);
  }
  return hipGetLastError();
}

template <typename real>
hipError_t launch_init(unsigned char* base, size_t slot_bytes, const void* E, const void* phi, int slots, int n,
                       int nplanes, unsigned* bad, hipStream_t st) {
  hipLaunchKernelGGL(k_init<real>, slot_grid(n, slots), dim3(256), 0, st, base, slot_bytes,
                     static_cast<const real*>(E), static_cast<const real*>(phi), n, nplanes, bad);
  return hipGetLastError();
}

hipError_t launch_upload(const void* pinned, void* dst, size_t bytes, hipStream_t st) {
  const int n = (int)(bytes / sizeof(int));
  hipLaunchKernelGGL(k_upload, dim3(std::min((n + 255) / 256, 64)), dim3(256), 0, st, static_cast<const int*>(pinned),
                     static_cast<int*>(dst), n);
  return hipGetLastError();
}

template <typename real>
hipError_t launch_op_setup(int* list, SlotCtl* ctl, SlotPtr<real>* optr, const SlotPtr<real>* ptrs, int s0, int count,
                           int listed, int phase, const void* in, size_t in_stride, void* out, size_t out_stride,
                           hipStream_t st) {
  hipLaunchKernelGGL(k_op_setup<real>, dim3(listed), dim3(64), 0, st, list, ctl, optr, ptrs, s0, count, listed, phase,
                     static_cast<const real*>(in), in_stride, static_cast<real*>(out), out_stride);
  return hipGetLastError();
}

template hipError_t launch_tick<float>(const LaunchGeom&, const TickBufs<float>&, int, hipStream_t, int);
template hipError_t launch_tick<double>(const LaunchGeom&, const TickBufs<double>&, int, hipStream_t, int);
template hipError_t launch_close<float>(const LaunchGeom&, const TickBufs<float>&, int, hipStream_t, int);
template hipError_t launch_close<double>(const LaunchGeom&, const TickBufs<double>&, int, hipStream_t, int);
template hipError_t launch_validate<float>(const float*, size_t, double, double, double, unsigned int*,
                                           hipStream_t);
template hipError_t launch_validate<double>(const double*, size_t, double, double, double, unsigned int*,
                                            hipStream_t);
#define SPFF_INSTANTIATE(R)                                                                                          \
  template hipError_t launch_fields<R>(const SlotPtr<R>*, const SlotParam*, const SlotCtl*, int, int, int,           \
                                       const FieldOut<R>&, hipStream_t);                                             \
  template hipError_t launch_state<R>(unsigned char*, size_t, size_t, size_t, size_t, int, int, const void*, void*,  \
                                      unsigned*, unsigned, unsigned*, hipStream_t);                                  \
  template hipError_t launch_init<R>(unsigned char*, size_t, const void*, const void*, int, int, int, unsigned*,     \
                                     hipStream_t);                                                                   \
  template hipError_t launch_op_setup<R>(int*, SlotCtl*, SlotPtr<R>*, const SlotPtr<R>*, int, int, int, int,         \
                                         const void*, size_t, void*, size_t, hipStream_t);
SPFF_INSTANTIATE(float)
SPFF_INSTANTIATE(double)
#undef SPFF_INSTANTIATE

// ===========================================================================
// Library-owned scratch of the allocation-free entry point
// (spff_load_step_static): one array per device, held until the process
// ends, shared by every call on that device.  In host code the array's name
// is not a device address; static_scratch() returns the address of the
// current device's copy, taken once per device with that device current.
// ===========================================================================
static __device__ __align__(256) unsigned char scratch[SPFF_STATIC_SCRATCH_BYTES];

hipError_t static_scratch(void** out) {
  constexpr int MAX_DEVICES = 64;
  static std::mutex mu;
  static void* addr[MAX_DEVICES] = {};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= MAX_DEVICES) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(mu);
  if (!addr[dev]) {
    void* ptr = nullptr;
    e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    addr[dev] = ptr;
  }
  *out = addr[dev];
  return hipSuccess;
}

}  // namespace spff
