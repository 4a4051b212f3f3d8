// launch_recorder.cpp -- the launchers and the HIP calls that the library's host code
// (api.cpp, plan.cpp) makes, as stubs that launch nothing and write one line per launch, so
// that the routes calls take can be tested without a GPU, for any number of compute units.
#include <hip/hip_runtime.h>

#include <cstdarg>
#include <cstdio>
#include <string>

#include "../paper_2607_28848_amd/csrc/kernels.h"

namespace {
std::string g_log;
int g_cus = 256;
alignas(256) char g_scratch[256];  // its address only: nothing is launched
hipEvent_t g_ev[2] = {};

hipError_t line(const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  g_log += buf;
  g_log += '\n';
  return hipSuccess;
}
template <class T>
T* fake() {
  return reinterpret_cast<T*>(g_scratch);
}
}  // namespace

extern "C" const char* recorder_log() { return g_log.c_str(); }
extern "C" void recorder_clear() { g_log.clear(); }
extern "C" void recorder_cus(int n) { g_cus = n; }
extern "C" const void* recorder_scratch() { return g_scratch; }

// ---- HIP ----
extern "C" {
hipError_t hipGetDevice(int* d) { return *d = 0, hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { return *v = g_cus, hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { return *e = fake<ihipEvent_t>(), hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { return *ms = 1.f, hipSuccess; }
hipError_t hipMemcpyAsync(void*, const void*, size_t, hipMemcpyKind, hipStream_t) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { return *s = fake<ihipStream_t>(), hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return line("wait_event"); }
}

namespace dsv {
hipError_t noalloc_scratch(void** out) { return *out = g_scratch, hipSuccess; }
void set_launch_events(hipEvent_t a, hipEvent_t b) { g_ev[0] = a, g_ev[1] = b; }
bool launch_events_pending() { return g_ev[0] || g_ev[1]; }
hipEvent_t take_launch_start() { return g_ev[0] = nullptr; }
hipEvent_t take_launch_stop() { return g_ev[1] = nullptr; }

static hipError_t tile(const char* nm, const GemmArgs& a, int tm, int tn) {
  set_launch_events(nullptr, nullptr);
  return line("%s tm=%d tn=%d M=%d Nout=%d C=%d tiles=%d whole=%d split=%d pieces=%d half=%d drop=%d", nm, tm, tn, a.M,
              a.Nout, a.C, a.n_mtiles * a.n_ntiles, a.dp_tiles, a.sk_tiles, a.sk_split, a.half_tiles, a.keep != nullptr);
}
hipError_t launch_gemm_nt(const GemmArgs& a, int tm, int tn, hipStream_t) { return tile("gemm_nt", a, tm, tn); }
hipError_t launch_gemm_nn(const GemmArgs& a, int tm, int tn, hipStream_t) { return tile("gemm_nn", a, tm, tn); }
hipError_t launch_gemm_group_nt(const GemmGroup& g, hipStream_t) {
  for (int p = 0; p < g.n; ++p) tile("group_nt", g.a[p], 256, 256);
  return hipSuccess;
}
hipError_t launch_gemm_group_nn(const GemmGroup& g, hipStream_t) {
  for (int p = 0; p < g.n; ++p) tile("group_nn", g.a[p], 256, 256);
  return hipSuccess;
}
hipError_t launch_part_gemm(const PartGroup& g, int cfg, int32_t, bool nn, hipStream_t) {
  take_launch_start();
  for (int p = 0; p < g.n; ++p) {
    const PartArgs& a = g.a[p];
    line("part cfg=%d nn=%d M=%d Nout=%d C=%d tiles=%d pieces=%d shrink=%d part=%zu bytes=%zu h_part=%zu h_bytes=%zu", cfg,
         nn, a.M, a.Nout, a.C, a.n_m * a.n_n, a.split, g.sh_off[p + 1] - g.sh_off[p], (size_t)a.part,
         (size_t)a.split * a.M * a.Nout * 4, (size_t)g.sh[p].part, (size_t)g.sh[p].pieces * g.T * g.r_max * 4);
  }
  return hipSuccess;
}
hipError_t launch_part_finish(FinishGroup g, int32_t n_items, int32_t, bool bwd, hipStream_t) {
  take_launch_stop();
  return line("finish n=%d items=%d bwd=%d drop=%d", g.n, n_items, bwd, g.a[0].keep != nullptr);
}
hipError_t launch_shrink(const SkinnyArgs&, int32_t n, int32_t, hipStream_t) { return line("shrink items=%d", n); }
hipError_t launch_shrink_train(const SkinnyArgs&, int32_t n, int32_t, hipStream_t) { return line("shrink_train items=%d", n); }
hipError_t launch_shrink_group(const SkinnyGroup&, int32_t n, int32_t, hipStream_t) { return line("shrink items=%d", n); }
hipError_t launch_shrink_train_group(const SkinnyGroup& g, int32_t n, int32_t, hipStream_t) {
  return g.n > 0 ? line("shrink_train items=%d", n) : hipSuccess;
}
hipError_t launch_gather_expand(const uint16_t*, int64_t, const uint16_t*, int32_t, int32_t, const int32_t*, int32_t n,
                                const int32_t*, const int32_t*, const float*, float*, hipStream_t) {
  return line("gather items=%d", n);
}
hipError_t launch_gather_group(const GatherGroup&, int64_t, int32_t, const int32_t*, int32_t n, const int32_t*,
                               const int32_t*, const float*, hipStream_t) {
  return n > 0 ? line("gather items=%d", n) : hipSuccess;
}
hipError_t launch_reduce_out(const ReduceOutArgs&, const ReduceOutArgs&, int32_t, int32_t, const int32_t*, int32_t,
                             const int32_t*, const int32_t*, const int32_t*, int32_t, hipStream_t) {
  return line("reduce_out");
}
hipError_t launch_reduce_out_group(const ReduceOutGroup&, int32_t, int32_t, const int32_t*, int32_t, const int32_t*,
                                   const int32_t*, const int32_t*, int32_t, hipStream_t) {
  return line("reduce_out");
}
hipError_t launch_token_reduce_group(const TokenReduceGroup&, int32_t, int32_t, hipStream_t) { return line("token_reduce"); }
hipError_t launch_g_finish_group(const SkinnyGroup&, int32_t, hipStream_t) { return line("g_finish"); }
hipError_t launch_adamw(const AdamWArgs&, int64_t, hipStream_t) { return line("adamw"); }
hipError_t launch_dropout_mask_group(const DropoutMaskGroup&, int32_t, hipStream_t) { return line("mask"); }
hipError_t launch_dropout_mask(uint32_t*, int32_t, int32_t, const DropoutSpec&, hipStream_t) { return line("mask"); }
hipError_t launch_f32_fwd(const F32Args&, hipStream_t) { return line("f32_fwd"); }
hipError_t launch_f32_bwd(const F32Args&, hipStream_t) { return line("f32_bwd"); }
}  // namespace dsv
