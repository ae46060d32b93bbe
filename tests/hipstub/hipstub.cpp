// A HIP runtime in host memory for tests of the library's host code without a
// device: the calls that libgdp2d.so makes are defined here and, as symbols of
// the executable, come before the real ones.  Copies and fills act at once,
// kernels do nothing, and a scenario (the argument) makes chosen calls fail
// and prints what it saw for the test to judge.
#include <hip/hip_runtime.h>
#include <dlfcn.h>
#include <errno.h>
#include <pthread.h>
#include <unistd.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <random>
#include <string>
#include <thread>
#include <vector>

#include "gdp2d.h"
#include "gdp_internal.h"

namespace {
std::mutex g_mu;
std::map<hipStream_t, int> g_pending;  // kernels launched on a stream since the host last waited for it
const std::thread::id g_main = std::this_thread::get_id();
const hipStream_t kUser = (hipStream_t)0x10;  // the stream of the caller's context
bool g_log_fills = false;
bool g_fail_launch = false;   // the next error query reports a failed launch
bool g_fail_threads = false;  // no thread can be created
bool g_fail_scratch = false;  // after the first allocation, every one until a batch's own buffers are made fails
int g_allocs = 0;
std::map<void *, size_t> g_live;  // allocations that have not been freed
}  // namespace

extern "C" {
int pthread_create(pthread_t *t, const pthread_attr_t *a, void *(*f)(void *), void *arg) {
  if (g_fail_threads) return EAGAIN;
  static const auto real = (int (*)(pthread_t *, const pthread_attr_t *, void *(*)(void *), void *))dlsym(RTLD_NEXT, "pthread_create");
  return real(t, a, f, arg);
}
hipError_t __hipPushCallConfiguration(dim3, dim3, size_t, hipStream_t) { return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3 *, dim3 *, size_t *shared, hipStream_t *) {
  *shared = 0;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void *, dim3, dim3, void **, size_t, hipStream_t) {
  std::lock_guard<std::mutex> g(g_mu);
  if (std::this_thread::get_id() == g_main) g_pending[kUser]++;
  return hipSuccess;
}
hipError_t hipGetLastError() {
  std::lock_guard<std::mutex> g(g_mu);
  if (g_fail_launch && g_pending[kUser]) {
    g_fail_launch = false;
    return hipErrorLaunchFailure;
  }
  return hipSuccess;
}
const char *hipGetErrorString(hipError_t) { return "scripted failure"; }
hipError_t hipGetDeviceCount(int *n) { *n = 1; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600 *p, int) {
  memset(p, 0, sizeof *p);
  p->multiProcessorCount = 256;
  return hipSuccess;
}
hipError_t hipGetSymbolAddress(void **p, const void *) { static char buf[1 << 20]; *p = buf; return hipSuccess; }
hipError_t hipMalloc(void **p, size_t n) {
  std::lock_guard<std::mutex> g(g_mu);
  if (g_fail_scratch && (std::this_thread::get_id() != g_main || ++g_allocs == 2)) return hipErrorOutOfMemory;
  *p = calloc(n, 1);
  g_live[*p] = n;
  return hipSuccess;
}
hipError_t hipFree(void *p) {
  std::lock_guard<std::mutex> g(g_mu);
  g_live.erase(p);
  free(p);
  return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t n, unsigned) {
  std::lock_guard<std::mutex> g(g_mu);
  *p = calloc(n, 1);
  g_live[*p] = n;
  return hipSuccess;
}
hipError_t hipHostFree(void *p) { return hipFree(p); }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind kind, hipStream_t) {
  memcpy(d, s, n);
  // a refinement has nothing left to do
  if (kind == hipMemcpyDeviceToHost && n == sizeof(gdp::DevState)) ((gdp::DevState *)d)->halt = gdp::kHaltDone;
  return hipSuccess;
}
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) { memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemsetAsync(void *d, int v, size_t n, hipStream_t) {
  memset(d, v, n);
  if (g_log_fills) printf("fill %d %zu\n", v & 0xff, n);
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t s) {
  std::lock_guard<std::mutex> g(g_mu);
  g_pending[s] = 0;
  return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) {
  std::lock_guard<std::mutex> g(g_mu);
  if (!g_fail_scratch) {  // (the launch scenario: the builders of a batch begin)
    printf("pending %d\n", g_pending[kUser]);
    fflush(stdout);
    _exit(0);
  }
  *s = (hipStream_t)0x20;
  return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipErrorNotSupported; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *) { return hipErrorNotSupported; }
hipError_t hipEventCreate(hipEvent_t *e) { *e = (hipEvent_t)0x30; return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipStreamSynchronize(kUser); }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { *ms = 0.f; return hipSuccess; }
}

namespace {
struct Input {
  std::vector<double> xy;
  std::vector<int32_t> seg{0, 1, 1, 2, 2, 3, 3, 0};
  gdp_pslg p;
  explicit Input(int n) : xy{0, 0, 1, 0, 1, 1, 0, 1} {
    std::mt19937 r(n);
    std::uniform_real_distribution<double> u(0.05, 0.95);
    for (int i = 0; i < 2 * n; i++) xy.push_back(u(r));
    memset(&p, 0, sizeof p);
    p.n_vertices = n + 4;
    p.n_segments = 4;
    p.xy = xy.data();
    p.seg = seg.data();
  }
};

// A batch that the library builds on the device (one input above the size of a
// workgroup build, the others below), or a small one that it builds on the host.
int batch(gdp_ctx *ctx, bool small = false) {
  std::vector<Input> in;
  in.emplace_back(Input(small ? 300 : 300000));
  for (int i = 0; i < 6; i++) in.emplace_back(Input((small ? 20 : 20000) + i));
  std::vector<gdp_pslg> ps;
  for (Input &x : in) ps.push_back(x.p), ps.back().xy = x.xy.data(), ps.back().seg = x.seg.data();
  const int n = (int)ps.size();
  std::vector<double> bsq(n, 2.0);
  std::vector<gdp_mesh *> out(n);
  std::vector<gdp_status> st(n);
  const gdp_status rc = gdp_refine_batch(ctx, ps.data(), bsq.data(), nullptr, n, out.data(), st.data(), nullptr);
  printf("batch %d\n", (int)rc);
  for (int i = 0; i < n && rc == GDP_OK && !small; i++) {
    int32_t want = 0;
    gdp_mesh_info info{};
    if (gdp_cdt_host(&ps[i], &want, 0, nullptr, nullptr, nullptr, nullptr, 0) != GDP_OK) return 1;
    if (out[i]) gdp_mesh_info_get(out[i], &info);
    printf("member %d %d %d\n", (int)st[i], info.n_triangles, want);
  }
  for (gdp_mesh *m : out) gdp_mesh_free(m);
  printf("live %zu\n", g_live.size());
  return 0;
}
}  // namespace

int main(int argc, char **argv) {
  const std::string what = argc > 1 ? argv[1] : "";
  gdp_ctx *ctx = nullptr;
  if (gdp_ctx_create(0, (void *)kUser, &ctx) != GDP_OK) return 1;
  if (what == "assign") {
    Input a(100), b(50);
    gdp_mesh *ma = nullptr, *mb = nullptr;
    if (gdp_mesh_create(ctx, &a.p, &ma) != GDP_OK || gdp_mesh_create(ctx, &b.p, &mb) != GDP_OK) return 1;
    g_log_fills = true;
    return gdp_mesh_assign(ctx, ma, mb) == GDP_OK ? 0 : 1;
  }
  if (what == "sizes") {
    for (int nv : {1000, 1000000, 67000000, 67200000, 89000000}) {
      gdp::DevCdtJob j{};
      j.nv = nv;
      printf("scratch %d %zu\n", nv, gdp::dev_cdt_batch_bytes(&j, 1));
    }
    return 0;
  }
  if (what == "launch") {
    g_fail_launch = true;
    return batch(ctx);
  }
  if (what == "threads") {
    g_fail_threads = true;
    if (batch(ctx, true)) return 1;
  }
  if (what == "scratch" || what == "threads") {
    g_fail_scratch = true;
    return batch(ctx);
  }
  return 1;
}
