// The tuner of vector plans, on the host: HIP calls over host memory, launches that only
// record.  fm_plan_tune must time the launch that a solve makes (the three components of a
// per-component pass at once, each device descriptor the component's own) and must leave
// the device descriptors equal to the plan's choices, also when an event call fails on the
// way.  Prints the launches looked at; exits non-zero on a mismatch.
#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>

#include "../../include/fluxmi.h"
#include "../../paper_2211_07777_amd/csrc/fm_pass.h"

static bool g_watch = false, g_solving = false;
static int g_r2r = 0, g_bad = 0, g_times = 0, g_fail_at = -1;

static void fail(const char* what) {
  std::fprintf(stderr, "mismatch: %s\n", what);
  ++g_bad;
}

// ---- HIP over host memory
extern "C" {
hipError_t hipMalloc(void** p, size_t n) { *p = std::calloc(n ? n : 1, 1); return *p ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipFree(void* p) { std::free(p); return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { return hipMalloc(p, n); }
hipError_t hipHostFree(void* p) { return hipFree(p); }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemsetAsync(void*, int, size_t, hipStream_t) { return hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t*, unsigned) { return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { *e = nullptr; return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { *e = nullptr; return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
// a different time for every sample, so that candidates win and lose
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) {
  *ms = 0.1f + 0.01f * (float)((++g_times * 37) % 101);
  return g_times == g_fail_at ? hipErrorUnknown : hipSuccess;
}
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* p, int) { std::memset(p, 0, sizeof(*p)); return hipSuccess; }
}

// ---- recorded launches
namespace fm {
static hipError_t look(const PassDesc& d, const PassDesc* dev) {
  if (!g_watch || d.kind != K_R2R) return hipSuccess;
  ++g_r2r;
  if (d.grid_y != 3) fail(g_solving ? "a solve launched one component" : "the tuner timed one component");
  if (std::memcmp(dev, &d, sizeof(d))) fail("the device descriptor is not the launched one");
  for (int q = 1; q < 3 && d.grid_y == 3; ++q) {
    if (dev[q].B != d.B || dev[q].tiles != d.tiles || dev[q].M != d.M || dev[q].r2r.half != d.r2r.half ||
        dev[q].lds_bytes != d.lds_bytes || dev[q].tw != d.tw)
      fail("a component's device descriptor has another tiling");
  }
  return hipSuccess;
}
template <typename T> hipError_t launch_pass(const PassDesc& d, const PassDesc* dev, const void*, void*, hipStream_t) { return look(d, dev); }
template <typename T> hipError_t launch_pass_batched(int, const PassDesc*, const int*, int, int, int, hipStream_t) { return hipSuccess; }
template <typename T> hipError_t launch_twiddles(void*, int, hipStream_t) { return hipSuccess; }
template <typename T> hipError_t launch_stage_twiddles(void*, int, hipStream_t) { return hipSuccess; }
template <typename T> hipError_t launch_wave_twiddles(void*, int, int, hipStream_t) { return hipSuccess; }
template <typename T> hipError_t launch_green_final(void*, const double*, const int[3], const int[3], const int[3], double, hipStream_t) { return hipSuccess; }
template <typename T> hipError_t launch_curl_real(const CurlReal&, hipStream_t) { return hipSuccess; }
hipError_t launch_green_sample(double*, const GreenGen&, hipStream_t) { return hipSuccess; }
hipError_t launch_lgf(double*, double*, double*, const LgfGen&, hipStream_t) { return hipSuccess; }
bool is_fast_len(int M) {
  for (int m : kFastLens)
    if (m == M) return true;
  return false;
}
#define FM_INST(T)                                                                                              \
  template hipError_t launch_pass<T>(const PassDesc&, const PassDesc*, const void*, void*, hipStream_t);        \
  template hipError_t launch_pass_batched<T>(int, const PassDesc*, const int*, int, int, int, hipStream_t);     \
  template hipError_t launch_twiddles<T>(void*, int, hipStream_t);                                              \
  template hipError_t launch_stage_twiddles<T>(void*, int, hipStream_t);                                        \
  template hipError_t launch_wave_twiddles<T>(void*, int, int, hipStream_t);                                    \
  template hipError_t launch_green_final<T>(void*, const double*, const int[3], const int[3], const int[3], double, hipStream_t); \
  template hipError_t launch_curl_real<T>(const CurlReal&, hipStream_t);
FM_INST(float)
FM_INST(double)
}  // namespace fm

int main() {
  // one and two symmetric axes; types I, II, III and semi-unbounded; fast and other lengths
  const int sets[][3][2] = {{{0, 0}, {3, 3}, {3, 3}}, {{0, 1}, {2, 2}, {3, 3}}, {{0, 0}, {1, 0}, {3, 3}}, {{0, 3}, {1, 1}, {2, 2}}};
  const int sizes[][3] = {{64, 64, 32}, {60, 48, 36}, {16, 128, 20}};
  int plans = 0;
  for (const auto& set : sets)
    for (const auto& n : sizes)
      for (int layout = 0; layout < 2; ++layout)
        for (int prec = 0; prec < 2; ++prec)
          for (int broken = 0; broken < 2; ++broken) {
            int bcv[3][3][2];
            for (int q = 0; q < 3; ++q)
              for (int a = 0; a < 3; ++a)
                for (int f = 0; f < 2; ++f) bcv[q][a][f] = (set[a][f] <= 1 && q == a) ? 1 - set[a][f] : set[a][f];
            const double h[3] = {0.1, 0.1, 0.1};
            fm_plan p = nullptr;
            g_watch = false;
            if (fm_plan_create_vector(&p, n, h, bcv, layout, 0, prec, 1, nullptr) != FM_OK) {
              fail("plan refused");
              continue;
            }
            ++plans;
            size_t bytes = 0;
            fm_plan_workspace_bytes(p, &bytes);
            void* ws = std::calloc(bytes, 1);
            g_watch = true;
            g_fail_at = broken ? g_times + 5 + 7 * layout : -1;
            const int rc = fm_plan_tune(p, ws, nullptr);
            if (rc != (broken ? FM_E_HIP : FM_OK)) fail("status of the tuner");
            g_solving = true;
            char io[8];
            if (fm_solve(p, io, io + 4, ws, nullptr) != FM_OK) fail("solve");  // launches are not run
            g_solving = false;
            fm_plan_destroy(p);
            std::free(ws);
          }
  std::printf("%d plans, %d real-to-real launches, %d mismatches\n", plans, g_r2r, g_bad);
  return g_bad || g_r2r < 100 ? 1 : 0;
}
