// A device for the host side of the library (lbm_ch_api.cpp) that runs on the CPU: the HIP
// calls and kernel launchers it uses, with device memory in host memory and every field
// reduced to its first value.  A population buffer or sum field holds the number of steps
// its state has taken, so that a state read from the wrong buffer, a step lost or made
// twice, and sums that no longer belong to their populations show as wrong numbers.
// Launches can be made to fail or to wait (those on one side stream), and are counted by
// kind.  Captured launches run when their graph is launched.
#include "device_double.h"

#include <stdlib.h>
#include <string.h>

#include <functional>
#include <map>
#include <vector>

#include "lbm_ch_internal.h"

namespace dbl {
int fail_in = -1;
std::map<std::string, int> count;
std::vector<Step> steps;
static std::vector<std::function<void()>>* capturing = nullptr;
std::function<float(const std::string&, int)> cost;  // us of a launch, for events
static float clock_us = 0.0f;

int source_device = 0;
hipStream_t side = nullptr;
std::vector<std::function<void()>> waiting;

static hipError_t enqueue(const char* kind, int shape, hipStream_t s, std::function<void()> f) {
  if (fail_in == 0) {
    fail_in = -1;
    return hipErrorLaunchFailure;
  }
  if (fail_in > 0) --fail_in;
  count[kind] += 1;
  if (cost) clock_us += cost(kind, shape);
  if (capturing) capturing->push_back(f);
  else if (side && s == side) waiting.push_back(f);
  else f();
  return hipSuccess;
}
static double get(const void* p) {
  double v;
  memcpy(&v, p, sizeof v);
  return v;
}
static void put(void* p, double v) { memcpy(p, &v, sizeof v); }
}  // namespace dbl

using dbl::enqueue;
using dbl::get;
using dbl::put;

extern "C" {
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { *p = calloc(1, n); return hipSuccess; }
hipError_t hipHostGetDevicePointer(void** d, void* h, unsigned) { *d = h; return hipSuccess; }
hipError_t hipHostFree(void* p) { free(p); return hipSuccess; }
hipError_t hipGetLastError(void) { return hipSuccess; }
hipError_t hipPointerGetAttributes(hipPointerAttribute_t* a, const void*) {
  memset(a, 0, sizeof *a);
  a->type = hipMemoryTypeDevice;
  a->device = dbl::source_device;
  if (dbl::source_device < 0) a->type = hipMemoryTypeHost;
  return dbl::source_device < -1 ? hipErrorInvalidValue : hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* from, size_t n, hipMemcpyKind, hipStream_t s) {
  return enqueue("copy", 0, s, [=] { memmove(d, from, n); });
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { *s = (hipStream_t)malloc(1); return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t s) { free(s); return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) {
  dbl::capturing = new std::vector<std::function<void()>>;
  return hipSuccess;
}
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g) {
  *g = (hipGraph_t)dbl::capturing;
  dbl::capturing = nullptr;
  return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t* x, hipGraph_t g, hipGraphNode_t*, char*, size_t) {
  *x = (hipGraphExec_t) new std::vector<std::function<void()>>(*(std::vector<std::function<void()>>*)g);
  return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t g) { delete (std::vector<std::function<void()>>*)g; return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t x) { delete (std::vector<std::function<void()>>*)x; return hipSuccess; }
hipError_t hipGraphLaunch(hipGraphExec_t x, hipStream_t s) {
  return enqueue("graph", 0, s, [=] { for (auto& f : *(std::vector<std::function<void()>>*)x) f(); });
}
hipError_t hipEventCreate(hipEvent_t* e) { *e = (hipEvent_t)calloc(1, sizeof(float)); return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t e) { free(e); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t) { *(float*)e = dbl::clock_us; return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t a, hipEvent_t b) {
  *ms = (*(float*)b - *(float*)a) * 1e-3f;
  return hipSuccess;
}
}

namespace lbmch {

uint32_t population_bytes(int storage, uint32_t pitch, uint32_t ny) {
  return (storage == 0 ? 36u : 20u) * pitch * ny;
}
bool march_ok(int vmode, int model, bool t1) {
  return t1 && (vmode == VEL_SEP || vmode == VEL_FIELD) && (model == 1 || model == 2);
}
bool phi_record_fused(bool walls, int vmode, int model, int storage) {
  return !walls && storage == 0 && vmode != VEL_NSFIELD && model < 3;
}
int phi_batch_blocks_per_cu(int, int, bool) { dbl::count["occupancy"] += 1; return 4; }
int diag_partial_blocks() { return 512; }
int rt_step_rows(int ty) { return ty >= 16 ? 16 : ty >= 8 ? 8 : ty >= 4 ? 4 : 2; }
hipError_t static_scratch_setup(int) { return hipSuccess; }
float* static_scratch(int) { return nullptr; }

static hipError_t population_step(const char* kind, int shape, StepArgs a, hipStream_t s) {
  return enqueue(kind, shape, s, [=] {
    if (a.phi_rec) *a.phi_rec = (float)get(a.src);
    dbl::steps.push_back({a.tf, 1});
    put(a.dst, get(a.src) + 1);
  });
}
hipError_t launch_phi_step(int tx, bool, int, int, int, const StepArgs& a, int, hipStream_t s) {
  return population_step("tile", tx * 1000 + a.ty, a, s);
}
hipError_t launch_phi_record(int tx, int, int, const StepArgs& a, int, hipStream_t s) {
  return population_step("record", tx * 1000 + a.ty, a, s);
}
hipError_t launch_pop_march(bool, int, int, int, const StepArgs& a, hipStream_t s) {
  return population_step("pop_march", a.mty, a, s);
}
hipError_t launch_phi_march(bool walls, int, int, int storage, bool to_g, int nt,
                            const StepArgs& a, hipStream_t s) {
  if ((walls && a.phi_rec) || (nt && (!to_g || storage != 0)) ||
      a.mstrips != march_strips(a.nx, a.mout))
    return hipErrorInvalidValue;
  return enqueue(nt ? "march_nt" : "march", a.mty, s, [=] {
    if (a.phi_rec) *a.phi_rec = (float)*a.msrc;
    dbl::steps.push_back({a.tf, 1});
    *a.mdst = *a.msrc + 1;
    if (to_g) put(a.dst, *a.mdst);
  });
}
hipError_t launch_phi_block(int rows, int, int, int, bool to_g, const StepArgs& a,
                            const BlockSteps& b, hipStream_t s) {
  if (b.steps < 1 || b.steps > BLOCK_STEPS) return hipErrorInvalidValue;
  return enqueue("block", rows * 10 + b.steps, s, [=] {
    for (int k = 0; k < b.steps; ++k) {
      if (a.phi_rec) a.phi_rec[(size_t)k * a.nx * a.ny] = (float)*a.msrc + k;
      dbl::steps.push_back({b.tf[k], 1});
    }
    *a.mdst = *a.msrc + b.steps;
    if (to_g) put(a.dst, *a.mdst);
  });
}
hipError_t launch_phi_single(int, int, int, const StepArgs& a, hipStream_t s) {
  return enqueue("single", 0, s, [=] {
    if (a.phi_rec) *a.phi_rec = (float)*a.msrc;
    dbl::steps.push_back({a.tf, 1});
    *a.mdst = *a.msrc + 1;
    put(a.dst, *a.mdst);
  });
}
hipError_t launch_march_batch(int, bool, bool to_g, const BatchArgs& b, hipStream_t s) {
  return enqueue("march_batch", 0, s, [=] {
    for (int i = 0; i < b.n; ++i) {
      const StepArgs& a = b.args[i];
      const double* src = b.parity ? a.mdst : a.msrc;
      double* dst = b.parity ? const_cast<double*>(a.msrc) : a.mdst;
      *dst = *src + 1;
      if (to_g) put(b.parity ? const_cast<void*>(a.src) : a.dst, *dst);
    }
  });
}
hipError_t launch_phi_batch(int tx, int, bool, bool persistent, const BatchArgs& b, int, hipStream_t s) {
  return enqueue("tile_batch", tx * 10 + persistent, s, [=] {
    for (int i = 0; i < b.n; ++i) {
      const StepArgs& a = b.args[i];
      const void* src = b.parity ? a.dst : a.src;
      put(b.parity ? const_cast<void*>(a.src) : a.dst, get(src) + 1);
    }
  });
}
hipError_t launch_ns_step(int, bool, int, const NsArgs&, int, hipStream_t) { return hipErrorInvalidValue; }
hipError_t launch_rt_step(int, bool, int, int, const StepArgs&, const float*, float*, int,
                          hipStream_t) { return hipErrorInvalidValue; }
hipError_t launch_init(bool, int, int, const Coef&, int, int, uint32_t, const float*, const float*,
                       const float*, const float*, const float*, const float*, const float*, float,
                       void* g, float*, hipStream_t s) {
  return enqueue("init", 0, s, [=] { put(g, 0.0); });
}
hipError_t launch_phi_field(bool, int, const void* g, uint32_t, int, int, float* phi, hipStream_t s) {
  return enqueue("phi_field", 0, s, [=] { *phi = (float)get(g); });
}
hipError_t launch_sum_field(bool, int, const void* g, uint32_t, int, int, double* m, hipStream_t s) {
  return enqueue("sum_field", 0, s, [=] { *m = get(g); });
}
hipError_t launch_load_sum(bool, int, const void* src, uint32_t, int, int, void* g, double* m,
                           hipStream_t s) {
  return enqueue("load_sum", 0, s, [=] {
    put(g, get(src));
    *m = get(src);
  });
}
hipError_t launch_phi_of_sum(const double* m, int64_t, float* phi, hipStream_t s) {
  return enqueue("phi_of_sum", 0, s, [=] { *phi = (float)*m; });
}
hipError_t launch_mu_field(bool, const Coef&, const float* phi, const double* m, int, int, float* mu, hipStream_t s) {
  return enqueue("mu", 0, s, [=] { *mu = m ? (float)*m : *phi; });
}
hipError_t launch_adjoint_step(const Coef&, float, int, int, int, const float*, const float*,
                               const float*, const float*, const float*, const float*, float,
                               const float*, const float*, float*, float*, float*, hipStream_t) {
  return hipErrorInvalidValue;
}
hipError_t launch_velocity_field(int, int, int, const float*, const float*, const float*,
                                 const float*, const float*, const float*, float, float*, float*,
                                 hipStream_t) { return hipErrorInvalidValue; }
hipError_t launch_fill(float*, float, int64_t, hipStream_t) { return hipSuccess; }
hipError_t launch_diag(bool, const Coef&, const float* phi, const double* m, const float*, int, int, double*,
                       double* out, hipStream_t s) {
  return enqueue("diag", 0, s, [=] {
    for (int i = 0; i < 8; ++i) out[i] = i == 7 ? 0.0 : m ? *m : *phi;
  });
}

}  // namespace lbmch
