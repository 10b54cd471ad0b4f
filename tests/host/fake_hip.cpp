#include "fake_hip.h"

#include <hip/hip_runtime.h>
#include <hipfft/hipfft.h>

#include <cstdlib>
#include <cstring>
#include <mutex>

namespace fake {
State& state() {
  static State s;
  return s;
}
static std::mutex mx;      // calls come from several threads
}  // namespace fake

using fake::state;

extern "C" {

hipError_t hipMalloc(void** p, size_t n) {
  std::lock_guard<std::mutex> lk(fake::mx);
  ++state().mallocs;
  *p = nullptr;
  if (n == state().fail_at) return hipErrorOutOfMemory;
  if (posix_memalign(p, 256, n ? n : 256)) return hipErrorOutOfMemory;
  std::memset(*p, 0, n);
  state().device[*p] = n;
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  std::lock_guard<std::mutex> lk(fake::mx);
  if (!p) return hipSuccess;
  if (!state().device.erase(p)) return hipErrorInvalidValue;
  std::free(p);
  return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
  std::lock_guard<std::mutex> lk(fake::mx);
  *p = nullptr;
  if (state().pinned_fails) return hipErrorOutOfMemory;
  *p = std::calloc(1, n);
  state().pinned[*p] = n;
  return hipSuccess;
}
hipError_t hipHostFree(void* p) {
  std::lock_guard<std::mutex> lk(fake::mx);
  if (!state().pinned.erase(p)) return hipErrorInvalidValue;
  std::free(p);
  return hipSuccess;
}
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) {
  state().copied_after = state().syncs;
  std::memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
  std::memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipMemset(void* d, int v, size_t n) {
  std::memset(d, v, n);
  return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t* e) { return hipEventCreateWithFlags(e, 0); }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
  std::lock_guard<std::mutex> lk(fake::mx);
  ++state().events;
  *e = reinterpret_cast<hipEvent_t>(std::malloc(1));
  return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t e) {
  std::lock_guard<std::mutex> lk(fake::mx);
  --state().events;
  std::free(e);
  return hipSuccess;
}
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) {
  *ms = 1.0f;
  return hipSuccess;
}
hipError_t hipEventQuery(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipGetDevice(int* d) {
  *d = 0;
  return hipSuccess;
}
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* p, int) {
  std::memset(p, 0, sizeof(*p));
  p->sharedMemPerBlock = 160 << 10;
  p->multiProcessorCount = 256;
  std::strcpy(p->gcnArchName, "gfx950");
  return hipSuccess;
}
const char* hipGetErrorString(hipError_t) { return "error"; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipGraphInstantiate(hipGraphExec_t* x, hipGraph_t, hipGraphNode_t*, char*, size_t) {
  *x = reinterpret_cast<hipGraphExec_t>(1);
  return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) {
  state().launches.push_back({"graph"});
  return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g) {
  *g = reinterpret_cast<hipGraph_t>(1);
  return hipSuccess;
}
hipError_t hipStreamCreate(hipStream_t* s) {
  *s = reinterpret_cast<hipStream_t>(1);
  return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) {
  ++state().syncs;
  return hipSuccess;
}
hipfftResult hipfftDestroy(hipfftHandle) { return HIPFFT_SUCCESS; }
hipfftResult hipfftExecD2Z(hipfftHandle, hipfftDoubleReal*, hipfftDoubleComplex*) { return HIPFFT_SUCCESS; }
hipfftResult hipfftPlanMany(hipfftHandle*, int, int*, int*, int, int, int*, int, int, hipfftType, int) {
  return HIPFFT_SUCCESS;
}
hipfftResult hipfftSetStream(hipfftHandle, hipStream_t) { return HIPFFT_SUCCESS; }

}  // extern "C"

namespace nflbm {

namespace {
hipError_t record(const char* kind, const StepArgs* a = nullptr) {
  fake::Launch l{kind};
  if (a) l.step = *a;
  std::lock_guard<std::mutex> lk(fake::mx);
  state().launches.push_back(l);
  return hipSuccess;
}
hipError_t record_fused(const FusedLaunch& f) {
  fake::Launch l{f.batch ? "fused2d_batch" : "fused2d"};
  if (f.one) l.fused = *f.one;
  l.shape = f;
  l.nsteps = f.nsteps;
  std::lock_guard<std::mutex> lk(fake::mx);
  state().launches.push_back(l);
  return hipSuccess;
}
hipError_t record_mob(int blocks, int nsteps) {
  fake::Launch l{"fused_mob"};
  l.nsteps = nsteps;
  l.shape.blocks = blocks;
  std::lock_guard<std::mutex> lk(fake::mx);
  state().launches.push_back(l);
  return hipSuccess;
}
}  // namespace

hipError_t launch_conc(int, int, int, const StepArgs& a, hipStream_t) { return record("conc", &a); }
hipError_t launch_update(int, int nc, int, const StepArgs& a, bool fields, hipStream_t) {
  if (fields)
    for (long long i = 0; i < (2 * nc + 7) * a.n; ++i) a.fields[i] = static_cast<double>(i);
  return record(fields ? "fields" : "update", &a);
}
hipError_t launch_init(int, int, int, const InitArgs&, hipStream_t) { return record("init"); }
hipError_t launch_batch_step(int, int, int, const BatchLaunch& b, hipStream_t) {
  record("batch", b.args);
  std::lock_guard<std::mutex> lk(fake::mx);
  state().launches.back().shape.blocks = b.blocks_update;
  return hipSuccess;
}
hipError_t launch_expand(int, int, int, const StepArgs&, hipStream_t) { return record("expand"); }
int groups_per_cu(int, int, int, const StepArgs&, bool) { return state().groups_per_cu; }
size_t conc_m_lds_bytes(int, int, int, int, bool) { return 32 << 10; }
hipError_t launch_expand_f(int, int, const StepArgs&, void*, hipStream_t) { return record("expand_f"); }
hipError_t launch_diag(int, int, int, const StepArgs&, int, double*, int* blocks, hipStream_t) {
  *blocks = 1;
  return record("diag");
}
hipError_t launch_lambda(const double*, double*, long long, hipStream_t) { return record("lambda"); }
hipError_t launch_spectrum(const void*, int, int, int, int, long long, int, double*, hipStream_t) {
  return record("spectrum");
}
int reduce_record_len(int N) { return 3 * N + 9; }
size_t update_lds_bytes(int, int, int, int) { return 32 << 10; }
hipError_t launch_build_bb(int, const unsigned char*, uint32_t*, const StepArgs&, hipStream_t) {
  return record("build_bb");
}
hipError_t launch_build_ob(int, int, uint32_t*, const StepArgs&, hipStream_t) { return record("build_ob"); }
hipError_t launch_outflow(int, int, int, const OutflowArgs&, hipStream_t) { return record("outflow"); }
hipError_t launch_mob_potentials(int, int, int, const MobArgs&, hipStream_t) { return record("mob_potentials"); }
hipError_t launch_mob_source(int, int, int, const MobArgs&, hipStream_t) { return record("mob_source"); }
hipError_t launch_fused2d_0(int, const FusedLaunch& f, hipStream_t) { return record_fused(f); }
hipError_t launch_fused2d_1(int, const FusedLaunch& f, hipStream_t) { return record_fused(f); }
hipError_t launch_fused2d_2(int, const FusedLaunch& f, hipStream_t) { return record_fused(f); }
hipError_t launch_fused_mob_0(int, const FusedMobArgs&, int blocks, int n, uint32_t, size_t, hipStream_t) {
  return record_mob(blocks, n);
}
hipError_t launch_fused_mob_1(int, const FusedMobArgs&, int blocks, int n, uint32_t, size_t, hipStream_t) {
  return record_mob(blocks, n);
}
hipError_t launch_fused_mob_2(int, const FusedMobArgs&, int blocks, int n, uint32_t, size_t, hipStream_t) {
  return record_mob(blocks, n);
}

}  // namespace nflbm
