// A stand-in for the GPU, to test the host driver (spff_api.cpp) on the CPU:
// the HIP calls that it makes, in host memory and in program order, and the
// launchers of spff_launch.hpp.  A "solver" step of slot s takes need[s]
// ticks; its control blocks, progress words, step queues and records are
// advanced as the row and closing kernels do.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "spff.h"
#include "spff_engine.hpp"
#include "spff_launch.hpp"

using namespace spff;

namespace {
struct State {
  std::vector<int> need;
  int fail_alloc = 0;             // fail the n-th pinned allocation from now
  int syncs = 0, rows = 0, cols = 0;
  unsigned all_flags = ~0u;       // flags that every pinned allocation had
  LaunchGeom geom{};              // of the last row kernel
} g;

int need_of(int s) { return s < (int)g.need.size() ? g.need[s] : 1; }

// the controller step of slot s after a tick
void controller(SlotCtl& c, int s, SlotSeq* seqs, StepRec* recs) {
  ++c.ticks;
  if (c.phase == PH_X_PROJ || c.phase == PH_X_LAP || c.phase == PH_X_DISP || c.ticks < need_of(s)) return;
  c.phase = PH_IDLE;
  c.t_start = 1000;
  c.t_end = 1000 + 100 * (uint64_t)c.ticks;
  if (!seqs || c.seq_pos >= seqs[s].len) return;
  StepRec r{};
  r.ticks = c.ticks;
  r.t_start = c.t_start;
  r.t_end = c.t_end;
  std::copy(c.eps_bar, c.eps_bar + 3, r.eps_bar);
  recs[(size_t)s * SEQ_MAX + c.seq_pos] = r;
  seqs[s].pos = ++c.seq_pos;
  if (c.seq_pos < seqs[s].len) {
    std::copy(seqs[s].eps_bar[c.seq_pos], seqs[s].eps_bar[c.seq_pos] + 3, c.eps_bar);
    c.phase = PH_M_RES;
    c.ticks = 0;
  }
}
}  // namespace

extern "C" {
void fake_reset() { g = State(); }
void fake_need(int slots, const int* ticks) { g.need.assign(ticks, ticks + slots); }
void fake_fail_alloc(int n) { g.fail_alloc = n; }
// counts since the last call: synchronisations, row kernels, column kernels
void fake_counts(int out[3]) {
  out[0] = g.syncs;
  out[1] = g.rows;
  out[2] = g.cols;
  g.syncs = g.rows = g.cols = 0;
}
unsigned fake_alloc_flags() { return g.all_flags; }
// kind, rows, threads of the row kernel and kind, columns, threads of the
// column kernel of the last tick
void fake_geom(int out[6]) {
  const LaunchGeom& G = g.geom;
  const int v[6] = {G.row_reg, G.R, G.threads, G.col_reg, G.W, G.threads_col};
  std::copy(v, v + 6, out);
}

hipError_t hipHostMalloc(void** p, size_t n, unsigned int flags) {
  g.all_flags &= flags;
  if (g.fail_alloc > 0 && --g.fail_alloc == 0) return hipErrorOutOfMemory;
  *p = std::calloc(1, n);
  return hipSuccess;
}
hipError_t hipHostFree(void* p) {
  std::free(p);
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
  std::memmove(d, s, n);
  return hipSuccess;
}
hipError_t hipMemcpy2DAsync(void* d, size_t dp, const void* s, size_t sp, size_t w, size_t h, hipMemcpyKind,
                            hipStream_t) {
  for (size_t i = 0; i < h; ++i) std::memcpy(static_cast<char*>(d) + i * dp, static_cast<const char*>(s) + i * sp, w);
  return hipSuccess;
}
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t) {
  std::memset(d, v, n);
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) {
  ++g.syncs;
  return hipSuccess;
}
hipError_t hipStreamQuery(hipStream_t) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t*, unsigned int) { return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipErrorNotSupported; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t*) { return hipErrorNotSupported; }
hipError_t hipGraphInstantiate(hipGraphExec_t*, hipGraph_t, hipGraphNode_t*, char*, size_t) {
  return hipErrorNotSupported;
}
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipErrorNotSupported; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipGetDevice(int* d) {
  *d = 0;
  return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) {
  *v = 100;  // clock: 100 kHz
  return hipSuccess;
}
const char* hipGetErrorString(hipError_t) { return "fake device error"; }
}  // extern "C"

namespace spff {

template <typename real>
hipError_t launch_tick(const LaunchGeom& G, const TickBufs<real>& B, int i, hipStream_t, int kernels) {
  if (kernels & TICK_COL) ++g.cols;
  if (!(kernels & TICK_ROW)) return hipSuccess;
  ++g.rows;
  g.geom = G;
  for (int k = 0; k < G.S; ++k) {
    const int s = B.list[k];
    if (s < 0) continue;
    SlotCtl c = B.ctl[i & 1][s];
    if (c.pending) controller(c, s, B.seqs, B.recs);
    c.pending = c.phase != PH_IDLE;
    ++c.tick_no;
    if (c.phase == PH_IDLE && c.idle_at == 0) c.idle_at = c.tick_no;
    if (B.post) B.post[s] = ((unsigned long long)c.idle_at << 32) | c.tick_no;
    B.ctl[(i & 1) ^ 1][s] = c;
  }
  return hipSuccess;
}

template <typename real>
hipError_t launch_close(const LaunchGeom& G, const TickBufs<real>& B, int k, hipStream_t, int slots) {
  for (int j = 0; j < (slots > 0 ? slots : G.S); ++j) {
    const int s = slots > 0 ? j : B.list[j];
    if (s < 0) continue;
    SlotCtl c = B.ctl[k & 1][s];
    if (c.pending) controller(c, s, B.seqs, B.recs);
    c.pending = 0;
    B.ctl[0][s] = c;
    if (B.mirror) B.mirror[s] = c;
  }
  return hipSuccess;
}

hipError_t launch_upload(const void* src, void* dst, size_t n, hipStream_t) {
  std::memcpy(dst, src, n);
  return hipSuccess;
}

#define FAKE(R)                                                                                                      \
  template hipError_t launch_tick<R>(const LaunchGeom&, const TickBufs<R>&, int, hipStream_t, int);                  \
  template hipError_t launch_close<R>(const LaunchGeom&, const TickBufs<R>&, int, hipStream_t, int);                 \
  template <>                                                                                                        \
  hipError_t launch_validate<R>(const R*, size_t, double, double, double, unsigned int*, hipStream_t) {              \
    return hipSuccess;                                                                                               \
  }                                                                                                                  \
  template <>                                                                                                        \
  hipError_t launch_fields<R>(const SlotPtr<R>*, const SlotParam*, const SlotCtl*, int, int, int,                    \
                              const FieldOut<R>&, hipStream_t) {                                                     \
    return hipSuccess;                                                                                               \
  }                                                                                                                  \
  template <>                                                                                                        \
  hipError_t launch_state<R>(unsigned char*, size_t, size_t, size_t, size_t, int, int, const void*, void*,           \
                             unsigned*, unsigned, unsigned* refused, hipStream_t) {                                  \
    *refused = 0;                                                                                                    \
    return hipSuccess;                                                                                               \
  }                                                                                                                  \
  template <>                                                                                                        \
  hipError_t launch_init<R>(unsigned char*, size_t, const void*, const void*, int, int, int, unsigned*,              \
                            hipStream_t) {                                                                           \
    return hipSuccess;                                                                                               \
  }                                                                                                                  \
  template <>                                                                                                        \
  hipError_t launch_op_setup<R>(int*, SlotCtl*, SlotPtr<R>*, const SlotPtr<R>*, int, int, int, int, const void*,     \
                                size_t, void*, size_t, hipStream_t) {                                                \
    return hipSuccess;                                                                                               \
  }
FAKE(float)
FAKE(double)
#undef FAKE

hipError_t static_scratch(void** out) {
  static void* p = std::aligned_alloc(256, SPFF_STATIC_SCRATCH_BYTES);
  *out = p;
  return hipSuccess;
}

}  // namespace spff
