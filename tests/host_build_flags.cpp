// The host runtime's build calls over stubbed HIP calls and kernel launches, in host memory (run by
// test_host_build_flags.py): no build's outcome may depend on what an earlier, failed build left in the context's
// flags.  The launches raise the flags that the kernels would; one HIP call can be made to fail.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "../include/ptraster.h"
#include "../paper_2204_01287_amd/csrc/internal.h"

namespace {
enum Call { NONE, COPY_BACK, SYNC, MEMSET };
Call g_fail = NONE;      // the next call of this kind fails, once
bool g_nonfinite = false;  // the cloud of the next launches holds a NaN

hipError_t outcome(Call c) {
  if (g_fail != c) return hipSuccess;
  g_fail = NONE;
  return hipErrorUnknown;
}
}  // namespace

extern "C" {
hipError_t hipGetDeviceCount(int* n) { return *n = 1, hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* p, int) {
  std::memset(p, 0, sizeof *p);
  std::strcpy(p->gcnArchName, "gfx950");
  return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { return *v = 256, hipSuccess; }
hipError_t hipMalloc(void** p, size_t n) { return *p = std::malloc(n), hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { return *p = std::malloc(n), hipSuccess; }
hipError_t hipFree(void* p) { return std::free(p), hipSuccess; }
hipError_t hipHostFree(void* p) { return std::free(p), hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return outcome(SYNC); }
const char* hipGetErrorString(hipError_t) { return "stub"; }
hipError_t hipMemsetAsync(void* p, int v, size_t n, hipStream_t) {
  const hipError_t e = outcome(MEMSET);
  if (e == hipSuccess) std::memset(p, v, n);
  return e;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind kind, hipStream_t) {
  const hipError_t e = kind == hipMemcpyDeviceToHost ? outcome(COPY_BACK) : hipSuccess;
  if (e == hipSuccess) std::memmove(d, s, n);
  return e;
}
}

namespace ptr {
int one(int) { return 1; }
#define SHAPE(W_, D_, T_)                                           \
  const RasterShape* PR_SHAPE_NAME_(W_, D_, T_)() {                 \
    static const RasterShape s = {W_, D_, T_, nullptr, nullptr, one}; \
    return &s;                                                      \
  }
PR_RASTER_SHAPES(SHAPE)
uint32_t accum_grid(int) { return 256; }
hipError_t static_work_init(int) { return hipSuccess; }
uint64_t small_scratch_bytes() { return 4096; }
uint64_t sort_scratch_bytes(uint64_t n) { return 64 * n; }
hipError_t launch_finite_check(const float*, uint64_t, uint32_t* flag, hipStream_t) {
  if (g_nonfinite) *flag |= 1u;
  return hipSuccess;
}
hipError_t launch_iota(uint32_t*, uint64_t, hipStream_t) { return hipSuccess; }
hipError_t launch_build_input(const BuildArgs& a, hipStream_t s) { return launch_finite_check(a.xyz, a.n, a.nonfinite, s); }
hipError_t launch_batch_bbox_spans(const float*, uint64_t, BatchRec*, hipStream_t) { return hipSuccess; }
hipError_t launch_quantize_spans(const float*, uint64_t, const BatchRec*, uint32_t*, uint32_t*, uint32_t*, hipStream_t) {
  return hipSuccess;
}
}  // namespace ptr

namespace {
int g_bad = 0;
void expect(const char* what, pr_status got, pr_status want) {
  if (got == want) return;
  std::printf("%s: status %d, expected %d (%s)\n", what, (int)got, (int)want, pr_last_error());
  g_bad++;
}

void* area(uint64_t n) { return std::aligned_alloc(256, (n + 511) / 256 * 256); }

pr_status build(pr_ctx* ctx, pr_cloud* cloud, bool spans, bool nonfinite, Call fail_at) {
  g_nonfinite = nonfinite;
  g_fail = fail_at;
  const uint32_t one_span[2] = {0, 100};
  const pr_status s = spans ? pr_build_batches_spans(ctx, cloud, one_span, nullptr, 1)
                            : pr_build_batches(ctx, cloud, 64, PR_ORDER_INPUT);
  g_fail = NONE;
  return s;
}
}  // namespace

int main() {
  pr_ctx* ctx = nullptr;
  expect("create", pr_create(0, nullptr, &ctx), PR_OK);
  const uint64_t n = 100;
  pr_cloud_bufs b{};
  expect("sizes", pr_cloud_sizes(n, 64, PR_ORDER_MORTON, &b.capacity), PR_OK);
  const pr_sizes& c = b.capacity;
  b.xyz = area(c.xyz), b.rgba = area(c.rgba), b.low = area(c.low), b.med = area(c.med), b.high = area(c.high);
  b.colors = area(c.colors), b.perm = area(c.perm), b.batches = area(c.batches), b.scratch = area(c.scratch);
  std::vector<float> xyz(3 * n, 0.f);
  std::vector<uint32_t> rgba(n, 0u);
  pr_cloud* cloud = nullptr;
  expect("load", pr_load_points(ctx, xyz.data(), rgba.data(), n, 0, &b, &cloud), PR_OK);
  for (bool spans : {false, true}) {
    expect("finite", build(ctx, cloud, spans, false, NONE), PR_OK);
    expect("non-finite", build(ctx, cloud, spans, true, NONE), PR_ENONFINITE);
    expect("finite after non-finite", build(ctx, cloud, spans, false, NONE), PR_OK);
    for (Call f : {COPY_BACK, SYNC, MEMSET}) {
      expect("non-finite, a HIP call fails", build(ctx, cloud, spans, true, f), PR_EDEVICE);
      expect("finite after the failed build", build(ctx, cloud, spans, false, NONE), PR_OK);
      expect("non-finite, a HIP call fails again", build(ctx, cloud, !spans, true, f), PR_EDEVICE);
      expect("non-finite after the failed build", build(ctx, cloud, spans, true, NONE), PR_ENONFINITE);
    }
  }
  pr_destroy(ctx);
  if (g_bad == 0) std::printf("host build flags ok\n");
  return g_bad ? 1 : 0;
}
