// Host-visible declarations of the kernel launchers defined in
// spff_kernels.hip (explicitly instantiated there for float and double).
#pragma once
#include <hip/hip_runtime.h>

#include "spff_engine.hpp"

namespace spff {

template <typename real> struct HostCplx;
template <> struct HostCplx<float> { using type = float2; };
template <> struct HostCplx<double> { using type = double2; };

struct LaunchGeom {
  int nx, ny, S;
  int R, ngr;  // rows per row work-group, row groups per slot
  int W, ngc;  // columns per column work-group, column groups per slot
  int threads;      // threads per row work-group
  int threads_col;  // threads per column work-group
  int col_reg;      // column kernel with register-resident transforms
  int col_pts;      // its points per lane: 8, or 16 (1024- and 2048-point columns)
  int row_reg;      // row kernels with register-resident transforms: 1 = 8, 2 = 4 points per lane
  int nyq_free;     // even grids: Nyquist modes of the strain fluctuation unconstrained
  size_t lds_row, lds_col;
};

// Device buffers of a handle's ticks.
template <typename real>
struct TickBufs {
  const int* list;            // listed slots (G.S entries, < 0: padding)
  const SlotPtr<real>* ptrs;  // per slot
  const SlotParam* prms;
  SlotCtl* ctl[2];            // control blocks; the host reads and writes ctl[0]
  const typename HostCplx<real>::type* twx;
  const typename HostCplx<real>::type* twy;
  double* prow[2];            // row partials, alternating by tick
  double* pcol;
  double* prof;               // per-slot byte counters, or null
  SlotSeq* seqs;              // device load-step queues, or null
  StepRec* recs;
  unsigned long long* post;   // progress words in pinned host memory, or null
  SlotCtl* mirror;            // host mirror of the control blocks, or null
  KTime* kt;                  // six timers (two ticks x three parts), or null
  unsigned long long* ktsum;  // folded times
};

// Tick i (0-based) of a run of ticks over the listed slots.  Tick 0 reads
// ctl[0], whose blocks must have no controller step pending (as the host
// and launch_close leave them).  kernels: which of the two to launch; the row
// kernel alone finishes the phase of tick i - 1.
enum { TICK_ROW = 1, TICK_COL = 2 };
template <typename real>
hipError_t launch_tick(const LaunchGeom& G, const TickBufs<real>& B, int i, hipStream_t st,
                       int kernels = TICK_ROW | TICK_COL);

// Closes a run of k ticks under one geometry: the controller step of tick
// k - 1, leaving the control blocks of the listed slots (slots > 0: of all
// `slots` slots) in ctl[0] and the mirror.
template <typename real>
hipError_t launch_close(const LaunchGeom& G, const TickBufs<real>& B, int k, hipStream_t st, int slots = 0);

template <typename real>
hipError_t launch_validate(const real* a, size_t n, double lo_excl, double lo_incl, double hi_incl,
                           unsigned int* bad, hipStream_t st);

// Caller buffers of the output fields ([slots][planes][n] each), null: not
// asked for.
template <typename real>
struct FieldOut {
  real *phi, *phi_ref, *strain, *stress, *psi, *eps;
};

// Output fields of slots s0 .. s0 + slots - 1.
template <typename real>
hipError_t launch_fields(const SlotPtr<real>* ptrs, const SlotParam* prms, const SlotCtl* ctls, int s0, int slots,
                         int n, const FieldOut<real>& O, hipStream_t st);

// State planes of all slots (byte offsets eps, phi, phi_ref in a slot) from
// `in` (real[slots][5][n]; nothing is copied if a value is not finite:
// *flag = token then, and *refused, in pinned host memory, tells), or to
// `out` if in is null.
template <typename real>
hipError_t launch_state(unsigned char* base, size_t slot_bytes, size_t eps, size_t phi, size_t phi_ref, int slots,
                        int n, const void* in, void* out, unsigned* flag, unsigned token, unsigned* refused,
                        hipStream_t st);

// First nplanes planes of every slot: E, phi, phi (null: zeros), zeros;
// counts bad values of E and phi in bad[0], bad[1].
template <typename real>
hipError_t launch_init(unsigned char* base, size_t slot_bytes, const void* E, const void* phi, int slots, int n,
                       int nplanes, unsigned* bad, hipStream_t st);

// bytes (a multiple of 4) from pinned host memory to the device
hipError_t launch_upload(const void* pinned, void* dst, size_t bytes, hipStream_t st);

// Control blocks, pointer table and list of a diagnostic operator over
// `count` slots from s0; in / out (elements per slot apart) take the place
// of the planes it reads and writes where they are not null.
template <typename real>
hipError_t launch_op_setup(int* list, SlotCtl* ctl, SlotPtr<real>* optr, const SlotPtr<real>* ptrs, int s0, int count,
                           int listed, int phase, const void* in, size_t in_stride, void* out, size_t out_stride,
                           hipStream_t st);

// Address of the current device's copy of the library-owned scratch array
// (SPFF_STATIC_SCRATCH_BYTES bytes, 256-byte aligned).
hipError_t static_scratch(void** out);

}  // namespace spff
