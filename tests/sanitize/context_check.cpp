// The host side of a solver context (rks_api.cpp) against a HIP runtime made of
// host memory with a budget: what a context does when device memory runs out
// in the middle of its life.  The launchers compute nothing; they check that
// the buffers they are given are allocated.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <map>
#include <vector>

#include "launch.hpp"
#include "rks.h"

static int failures = 0;
#define CHECK(c)                                  \
  do {                                            \
    if (!(c)) {                                   \
      std::printf("line %d: %s\n", __LINE__, #c); \
      ++failures;                                 \
    }                                             \
  } while (0)

// ---- the runtime ---------------------------------------------------------------
static std::map<const char*, size_t> live;
static size_t room = (size_t)1 << 40;
static hipError_t last = hipSuccess;

static bool allocated(const void* p, size_t bytes = 1) {
  auto it = live.upper_bound((const char*)p);
  if (it == live.begin()) return false;
  --it;
  return (const char*)p + bytes <= it->first + it->second;
}

extern "C" {
hipError_t hipMalloc(void** p, size_t bytes) {
  if (bytes > room) return last = hipErrorOutOfMemory;
  *p = std::calloc(bytes, 1);
  live[(char*)*p] = bytes;
  room -= bytes;
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  auto it = live.find((char*)p);
  CHECK(it != live.end());
  room += it->second;
  live.erase(it);
  std::free(p);
  return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t bytes, unsigned) { return (*p = std::calloc(bytes, 1)) ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipHostFree(void* p) { std::free(p); return hipSuccess; }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { std::memmove(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) { std::memmove(d, s, n); return hipSuccess; }
hipError_t hipMemset(void* d, int v, size_t n) { std::memset(d, v, n); return hipSuccess; }
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t) { std::memset(d, v, n); return hipSuccess; }
hipError_t hipMemGetInfo(size_t* f, size_t* t) { *f = *t = room; return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipGetLastError() { hipError_t e = last; last = hipSuccess; return e; }
const char* hipGetErrorString(hipError_t) { return "error"; }
hipError_t hipEventCreate(hipEvent_t*) { return hipErrorUnknown; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float*, hipEvent_t, hipEvent_t) { return hipErrorUnknown; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { *s = (hipStream_t)&live; return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }

// A recorded graph is the list of what its launches do.
typedef std::vector<std::function<void()>> Graph;
static Graph* recording = nullptr;
static int replays = 0;
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { recording = new Graph; return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g) { *g = (hipGraph_t)recording; recording = nullptr; return hipSuccess; }
hipError_t hipGraphInstantiate(hipGraphExec_t* x, hipGraph_t g, hipGraphNode_t*, char*, size_t) {
  *x = (hipGraphExec_t) new Graph(*(Graph*)g);
  return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t g) { delete (Graph*)g; return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t x) { delete (Graph*)x; return hipSuccess; }
hipError_t hipGraphLaunch(hipGraphExec_t x, hipStream_t) {
  for (auto& f : *(Graph*)x) f();
  ++replays;
  return hipSuccess;
}
}  // extern "C"

static void run(std::function<void()> f) {
  if (recording) recording->push_back(f);
  else f();
}
static void use(const void* p, size_t bytes = 1) {
  if (p) run([=] { CHECK(allocated(p, bytes)); });
}

// ---- the launchers ---------------------------------------------------------------
static int resid_cols = 0;  // scratch columns of the last residual launch
static int stored = 0, evaluated = 0;  // Gaussian sketches
namespace rks {
int launch_spmv_sketch(const LaunchEnv& e, const void* x, void* w, double*, int, int) { use(x); use(w); return 1; }
int launch_gauss(const LaunchEnv& e, const void*, const void*, double*, double*) {
  use(e.om);
  run([om = e.om] { (om ? stored : evaluated) += 1; });
  return 1;
}
void launch_omega_fill(const LaunchEnv& e, double* om) { use(om, (size_t)(e.sp.d + 1) / 2 * e.n * 16); }
void launch_reduce(const LaunchEnv&, const double*, int, const double*, int, double*, double*) {}
static void column(const LaunchEnv& e, int t, double* S, double* cs) {
  run([=, d = e.sp.d] { S[t + (size_t)t * d] = cs[t] = 1.0; });
}
void launch_ls(const LaunchEnv& e, int t, int, int, const double*, const double*, double* S, double*, int, double*, double* cs, double*, double*, int*, double) { column(e, t, S, cs); }
int launch_update(const LaunchEnv&, int, const void*, int64_t, const void*, const double*, const double*, const double*, double*, int, void*, double*) { return 1; }
int launch_ls_update(const LaunchEnv& e, int t, int, const double*, const double*, double* S, double* B, int ldb, double*, double* cs, double*, double*, int*, double, const void* U, int64_t, const void* w, void* u, double*) {
  use(U);
  use(w);
  use(u);
  column(e, t, S, cs);
  run([=] {
    static int calls = 0;
    B[t + (size_t)t * ldb] = 1.0 + 0.01 * ++calls;
    B[t + 1 + (size_t)t * ldb] = 0.001;
  });
  return 1;
}
int launch_init(const LaunchEnv&, void* u, const double*, uint32_t, uint32_t, double*, int, int, uint32_t, uint32_t) { use(u); return 1; }
void launch_rotate(const LaunchEnv&, const void* U, int64_t, int, int, void* O, int64_t, int, int, const double*, int, int, double, int) { use(U); use(O); }
int launch_resid(const LaunchEnv& e, int64_t, const double* X, int ke, const int*, const double*, const double*, double* Xi, int xcols, double* part) {
  use(X, (size_t)e.n * ke * 8);
  if (!e.sl) use(Xi, (size_t)e.n * xcols * 8);
  use(part, (size_t)kResidMaxG * 2 * ke * 8);
  resid_cols = xcols;
  return 1;
}
void launch_normalise(const LaunchEnv&, double*, int, const int*, const double*) {}
void launch_copy16(hipStream_t, const void*, void*, int64_t) {}
void launch_read16(hipStream_t, const void*, int64_t) {}
int launch_dots(const LaunchEnv&, int, const void*, int64_t, const void*, double*) { return 1; }
void launch_reduce_len(const LaunchEnv&, const double*, int, double*, int) {}
void launch_ks_finalize(const LaunchEnv&, int, const double*, const double*, int, double*, int, double*, int*, double) {}
void launch_ks_start(const LaunchEnv&, const double*, double*) {}
int scratch_address(double**) { return 1; }
int launch_sketch_scratch(const LaunchEnv&, const double*, double*, double*) { return 1; }
}  // namespace rks

// ---- contexts ---------------------------------------------------------------------
static const int64_t n = 4096;
static const int k = 8, m = 24, d = 60;
static const size_t col = n * 8, xr = col * (k + 1), rpart = (size_t)(k + 1) * 2 * (rks::kResidMaxG + 1) * 8,
                    u64 = col * (m + 1);

static rks_ctx* context(void (*set)(rks_opts*)) {
  std::vector<int32_t> rp(n + 1), ci(n);
  std::vector<double> v(n);
  for (int64_t i = 0; i < n; ++i) rp[i + 1] = (int32_t)i + 1, ci[i] = (int32_t)i, v[i] = 1.0 + i;
  rks_csr A{n, n, rp.data(), ci.data(), v.data(), 0};
  rks_opts o;
  rks_opts_default(&o);
  o.spmv_layout = RKS_SPMV_ROWS;
  o.max_restarts = 3;
  set(&o);
  rks_ctx* c = nullptr;
  CHECK(rks_create(&A, k, m, d, RKS_LM, 1e-10, &o, &c) == RKS_OK);
  return c;
}

static int eigpairs(rks_ctx* c) {
  std::vector<double> re(k + 1), im(k + 1), res(k + 1);
  return rks_eigpairs(c, re.data(), im.data(), nullptr, 0, res.data());
}

// The residuals' scratch: eight columns, two where there is no room for them.
static void residual_scratch() {
  for (int fits : {8, 2, 0}) {
    rks_ctx* c = context([](rks_opts*) {});
    CHECK(rks_solve(c, nullptr, 0, nullptr) == RKS_ENOTCONV);
    room = xr + rpart + (fits ? fits * col : col);
    CHECK(eigpairs(c) == (fits ? RKS_OK : RKS_ENOMEM));
    CHECK(!fits || resid_cols == fits);
    CHECK(hipGetLastError() == hipSuccess);
    room = (size_t)1 << 40;
    CHECK(eigpairs(c) == RKS_OK);
    rks_destroy(c);
    CHECK(live.empty());
  }
  // the FP64 basis of the refinement, after the wide scratch of the first phase
  rks_ctx* c = context([](rks_opts* o) { o->precision = RKS_PREC_V32; });
  room = xr + rpart + 2 * col + u64;
  CHECK(rks_solve(c, nullptr, 0, nullptr) == RKS_ENOTCONV);
  CHECK(eigpairs(c) == RKS_OK && resid_cols == 2);
  room = (size_t)1 << 40;
  rks_destroy(c);
  CHECK(live.empty());
}

static void gauss(rks_opts* o) {
  o->sketch_kind = RKS_SKETCH_GAUSS;
  o->graphs = 1;
}

// Omega is not stored on request, nor where it would take more than 1/32 of the
// memory that the context's own buffers leave.
static void omega_left_out() {
  const size_t om = (size_t)(d + 1) / 2 * n * 16, before = room;
  rks_ctx* c = context(gauss);
  const size_t taken = before - room - om;
  rks_destroy(c);
  for (int kind = 0; kind < 3; ++kind) {
    stored = evaluated = 0;
    room = kind == 0 ? room : taken + 32 * om - (kind == 1 ? 32 : 0);
    c = kind == 0 ? context([](rks_opts* o) { gauss(o); o->omega = RKS_OMEGA_EVALUATE; }) : context(gauss);
    CHECK(rks_solve(c, nullptr, 0, nullptr) == RKS_ENOTCONV);
    CHECK(kind == 2 ? stored > 0 && evaluated == 0 : stored == 0 && evaluated > 0);
    rks_destroy(c);
    room = (size_t)1 << 40;
  }
}

// A stored Omega gives way to what a context allocates at its first use.
static void stored_omega() {
  rks_ctx* c = context(gauss);
  CHECK(rks_solve(c, nullptr, 0, nullptr) == RKS_ENOTCONV);
  CHECK(rks_solve(c, nullptr, 0, nullptr) == RKS_ENOTCONV && replays > 0);
  CHECK(stored > 0 && evaluated == 0);
  room = xr - 8;
  CHECK(eigpairs(c) == RKS_OK);
  stored = 0;
  CHECK(rks_solve(c, nullptr, 0, nullptr) == RKS_ENOTCONV && eigpairs(c) == RKS_OK);  // no graph reads it
  CHECK(stored == 0 && evaluated > 0);
  room = (size_t)1 << 40;
  rks_destroy(c);
  CHECK(live.empty());
  // in the middle of a solve: the FP64 basis of the refinement
  evaluated = 0;
  c = context([](rks_opts* o) { gauss(o); o->precision = RKS_PREC_V32; });
  room = xr + rpart + u64 - 8;
  CHECK(rks_solve(c, nullptr, 0, nullptr) == RKS_ENOTCONV && evaluated > 0);
  CHECK(eigpairs(c) == RKS_OK);
  room = (size_t)1 << 40;
  rks_destroy(c);
  CHECK(live.empty());
}

int main() {
  residual_scratch();
  stored_omega();
  omega_left_out();
  std::printf("ok: %d failures\n", failures);
  return failures != 0;
}
