// Lifetimes of handles and batches in the library's host code, on the CPU: dg_host.cpp and dg_batch.cpp with
// stand-ins for the HIP calls and the kernel launches.  Freed memory is overwritten, device allocations are counted,
// and every stream and event that reaches a HIP call has to be a live one.
#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <set>
#include <vector>

#include <malloc.h>

#include "../paper_1910_02858_amd/csrc/dg_internal.h"

void *operator new(size_t n) {
  if (void *p = std::malloc(n ? n : 1)) return p;
  throw std::bad_alloc();
}
void operator delete(void *p) noexcept {
  for (size_t i = 0, n = p ? malloc_usable_size(p) : 0; i < n; ++i) ((volatile unsigned char *)p)[i] = 0xdd;
  std::free(p);
}
void operator delete(void *p, size_t) noexcept { operator delete(p); }

static std::set<void *> streams, device;
static int bad = 0;
static hipError_t live(hipStream_t s) {
  if (s && !streams.count(s)) { ++bad; std::printf("a call on a stream that is not live\n"); }
  return hipSuccess;
}

extern "C" {
hipError_t hipMalloc(void **p, size_t n) { *p = std::calloc(n, 1); device.insert(*p); return hipSuccess; }
hipError_t hipFree(void *p) {
  if (p && !device.erase(p)) { ++bad; std::printf("freed twice\n"); return hipSuccess; }
  std::free(p);
  return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { return hipMalloc(p, n); }
hipError_t hipHostFree(void *p) { return hipFree(p); }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind k, hipStream_t st) { live(st); return hipMemcpy(d, s, n, k); }
hipError_t hipMemset(void *d, int c, size_t n) { std::memset(d, c, n); return hipSuccess; }
hipError_t hipMemsetAsync(void *d, int c, size_t n, hipStream_t st) { live(st); return hipMemset(d, c, n); }
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { *s = (hipStream_t)std::malloc(8); streams.insert(*s); return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t s) { live(s); streams.erase(s); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s) { return live(s); }
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t, unsigned) { return live(s); }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { *e = (hipEvent_t)std::malloc(8); return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *e) { return hipEventCreateWithFlags(e, 0); }
hipError_t hipEventDestroy(hipEvent_t e) { std::free(e); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t s) { return live(s); }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *t, hipEvent_t, hipEvent_t) { *t = 1.f; return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t s, hipStreamCaptureMode) { return live(s); }
hipError_t hipStreamEndCapture(hipStream_t s, hipGraph_t *g) { *g = (hipGraph_t)std::malloc(8); return live(s); }
hipError_t hipGraphDestroy(hipGraph_t g) { std::free(g); return hipSuccess; }
hipError_t hipGraphInstantiate(hipGraphExec_t *e, hipGraph_t, hipGraphNode_t *, char *, size_t) { *e = (hipGraphExec_t)std::malloc(8); return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t e) { std::free(e); return hipSuccess; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t s) { return live(s); }
}

namespace dg {
int static_scratch_setup(int) { return DG_OK; }
int launch_final_reduce(int, const double *, int, double *, hipStream_t) { return DG_OK; }
int launch_axpby(double *, const double *, double, double, size_t, hipStream_t) { return DG_OK; }
int launch_mass(const double *, const double *, int, size_t, double *, hipStream_t) { return DG_OK; }
int fused_epb(int N, bool) { return N <= 7 ? 1 : 0; }
int launch_fused_lift(const FusedView &, hipStream_t) { return DG_OK; }
int launch_fused_split(const FusedView &, bool, int, hipStream_t) { return DG_OK; }
#define LAUNCH(NAME, ...) template <int N> int NAME(__VA_ARGS__) { return DG_OK; }
LAUNCH(launch_prolong, const Geo &, const Phys &, const double *, hipStream_t)
LAUNCH(launch_lift, const Geo &, const Phys &, bool, int, const double *, double *, double *, hipStream_t)
LAUNCH(launch_main, const Geo &, const Phys &, bool, int, int, const double *, const double *, double *, double *, double, double, double, int, hipStream_t)
LAUNCH(launch_vjp, const Geo &, const Phys &, int, int, bool, const double *, const double *, double *, const double *, double *, double, int, double *, double, double, hipStream_t)
LAUNCH(launch_reduce, const Geo &, const Phys &, int, const double *, double *, hipStream_t)
LAUNCH(launch_fv_face, const Geo &, const Phys &, const FvGeo &, bool, const double *, hipStream_t)
LAUNCH(launch_fv_volume, const Geo &, const Phys &, const FvGeo &, const double *, double *, double *, double, double, double, int, hipStream_t)
LAUNCH(launch_fv_switch, const Geo &, const Phys &, const FvGeo &, double *, int, hipStream_t)
LAUNCH(launch_fv_lists, const Geo &, const FvGeo &, hipStream_t)
LAUNCH(launch_mortar_lift, const Geo &, const Phys &, bool, const MortarDesc *, int, const double *, hipStream_t)
LAUNCH(launch_mortar_flux, const Geo &, const Phys &, bool, int, const MortarDesc *, int, const double *, const double *, hipStream_t)
LAUNCH(launch_batch_lift, const BatchView &, int, hipStream_t)
LAUNCH(launch_batch_split, const BatchView &, bool, int, int, hipStream_t)
}  // namespace dg

// the launches are defined above, so the sources below instantiate them where they call them
#include "../paper_1910_02858_amd/csrc/dg_host.cpp"
#define aligned8 batch_aligned8  // both sources have one
#include "../paper_1910_02858_amd/csrc/dg_batch.cpp"

static dg_handle *make(int N, int k, hipStream_t st) {
  const int n = N + 1, K = k * k * k, n3 = n * n * n;
  double x[16], w[16];
  dg_nodes(N, DG_NODES_LGL, x, w);
  std::vector<double> X((size_t)K * 3 * n3);
  std::vector<int32_t> nb(6 * K);
  std::vector<int8_t> sd(6 * K);
  for (int e = 0; e < K; ++e) {
    const int c[3] = {e % k, e / k % k, e / k / k};
    for (int q = 0; q < n3; ++q) {
      const int id[3] = {q % n, q / n % n, q / n / n};
      for (int d = 0; d < 3; ++d) X[((size_t)e * 3 + d) * n3 + q] = c[d] + 0.5 * (x[id[d]] + 1);
    }
    for (int s = 0; s < 6; ++s) {
      int g[3] = {c[0], c[1], c[2]};
      g[s / 2] = (g[s / 2] + ((s & 1) ? 1 : k - 1)) % k;
      nb[6 * e + s] = g[0] + k * (g[1] + k * g[2]);
      sd[6 * e + s] = (int8_t)(s ^ 1);
    }
  }
  dg_mesh m{};
  m.n_elems = K; m.n_geo = N; m.xgeo = X.data(); m.nbr_elem = nb.data(); m.nbr_side = sd.data();
  dg_scheme sc{};
  sc.eqn = DG_NAVIER_STOKES; sc.form = DG_FORM_SPLIT; sc.volflux = DG_VF_KEP; sc.riemann = DG_RS_ROE;
  sc.gamma = 1.4; sc.R = 1.0; sc.mu = 1e-3; sc.Pr = 0.72;
  dg_handle *h = nullptr;
  if (dg_init(&m, N, DG_NODES_LGL, &sc, st, &h)) { ++bad; std::printf("dg_init failed\n"); }
  return h;
}

int main() {
  for (int order = 0; order < 3; ++order) {  // members last, members first, one member before and one after
    hipStream_t st;
    hipStreamCreateWithFlags(&st, 0);
    dg_handle *h[2] = {make(2, 2, st), make(3, 1, st)};
    dg_batch *b = nullptr;
    if (dg_batch_create(h, 2, &b)) { ++bad; std::printf("dg_batch_create failed\n"); }
    std::vector<double> a[2][3];
    double *p[3][2];
    for (int i = 0; i < 2; ++i)
      for (int j = 0; j < 3; ++j) {
        a[i][j].resize((size_t)h[i]->K * 5 * h[i]->n3);
        p[j][i] = a[i][j].data();
      }
    const double dt[2] = {1e-3, 1e-3};
    if (dg_batch_step(b, p[0], p[1], p[2], dt, 1) || dg_batch_step(b, p[0], p[1], p[2], dt, 0)) { ++bad; std::printf("dg_batch_step failed\n"); }
    if (order) dg_destroy(h[0]);
    if (order == 1) dg_destroy(h[1]);
    dg_batch_destroy(b);
    if (!order) dg_destroy(h[0]);
    if (order != 1) dg_destroy(h[1]);
    hipStreamDestroy(st);
    if (!device.empty() || !streams.empty()) { ++bad; std::printf("order %d: %zu allocations, %zu streams left\n", order, device.size(), streams.size()); }
  }
  // a batch that is refused leaves its members as they were
  dg_handle *h = make(1, 1, nullptr), *twice[2] = {h, h};
  dg_batch *b = nullptr;
  if (dg_batch_create(twice, 2, &b) != DG_ERR_ARG || b) { ++bad; std::printf("a member listed twice was accepted\n"); }
  dg_destroy(h);
  if (!device.empty()) { ++bad; std::printf("the refused batch's member was not freed\n"); }
  std::printf(bad ? "FAILED\n" : "ok\n");
  return bad ? 1 : 0;
}
