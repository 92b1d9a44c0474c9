// staging.h on the host alone: the HIP calls it makes are defined here.  A
// "device" copy is a memcpy; each call is checked against the rules that the
// real one follows (a thread's own meaning of the per-thread stream, one
// device per thread), and host failures are brought about on request.
// Usage: staging_host <case>; exit status 0 when the case holds.
#include "../paper_2411_14631_amd/csrc/staging.h"

#include <cstdio>
#include <cstdlib>
#include <new>
#include <string>
#include <vector>

namespace {
std::atomic<int> g_copies{0}, g_foreign{0};   // copies asked for; those by another thread than the caller's
const std::thread::id g_main = std::this_thread::get_id();
thread_local int t_device = 0;
bool g_refuse_alloc = false;           // operator new throws
std::vector<double> g_pinned;          // the host memory known to the runtime
}  // namespace

void* operator new(std::size_t n) {
  void* p = g_refuse_alloc ? nullptr : std::malloc(n);
  if (!p) throw std::bad_alloc();
  return p;
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, std::size_t) noexcept { std::free(p); }

extern "C" {
hipError_t hipMemcpyAsync(void* dst, const void* src, size_t n, hipMemcpyKind, hipStream_t) {
  std::memcpy(dst, src, n);
  ++g_copies;
  if (std::this_thread::get_id() != g_main) ++g_foreign;
  return t_device == 3 ? hipSuccess : hipErrorInvalidDevice;
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
  *e = reinterpret_cast<hipEvent_t>(std::malloc(1));
  return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t e) {
  std::free(e);
  return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
  *p = std::malloc(n);
  return hipSuccess;
}
hipError_t hipHostFree(void* p) {
  std::free(p);
  return hipSuccess;
}
hipError_t hipGetDevice(int* d) {
  *d = t_device;
  return hipSuccess;
}
hipError_t hipSetDevice(int d) {
  t_device = d;
  return hipSuccess;
}
hipError_t hipGetLastError(void) { return hipSuccess; }
// memory the runtime does not know is an error, as some versions report it
hipError_t hipPointerGetAttributes(hipPointerAttribute_t* a, const void* p) {
  std::memset(a, 0, sizeof *a);
  const auto* d = static_cast<const double*>(p);
  if (!g_pinned.empty() && d >= g_pinned.data() && d < g_pinned.data() + g_pinned.size()) {
    a->type = hipMemoryTypeHost;
    return hipSuccess;
  }
  return hipErrorInvalidValue;
}
}

int main(int argc, char** argv) {
  if (argc < 2) return 2;
  const std::string what = argv[1];
  t_device = 3;
  // five rows of 2.5 MB, a gap between them on the device
  constexpr int kRows = 5;
  constexpr size_t kRow = 327680 + 3, kStride = kRow + 17;
  std::vector<double> dev(kRows * kStride), host(kRows * kRow, -1.0);
  for (size_t i = 0; i < dev.size(); ++i) dev[i] = double(i);
  double* out = host.data();
  hipStream_t st = reinterpret_cast<hipStream_t>(std::malloc(1));
  if (what == "per_thread_stream") st = hipStreamPerThread;
  if (what == "pinned") {
    g_pinned.assign(kRows * kRow, -1.0);
    out = g_pinned.data();
  }
  ry::Staging s;
  g_refuse_alloc = what == "no_host_memory";
  const hipError_t e = s.download(out, dev.data(), sizeof(double) * kRow, sizeof(double) * kStride, kRows, st);
  g_refuse_alloc = false;
  s.release();
  if (e != hipSuccess) return std::printf("status %d\n", int(e)), 1;
  for (int r = 0; r < kRows; ++r)
    for (size_t i = 0; i < kRow; ++i)
      if (out[r * kRow + i] != dev[r * kStride + i]) return std::printf("row %d value %zu\n", r, i), 1;
  if (what != "pageable" && g_foreign) return std::printf("%d copies by other threads\n", int(g_foreign)), 1;
  if (what == "pageable" && g_copies <= kRows) return std::printf("%d copies\n", int(g_copies)), 1;
  if (what == "pinned" && g_copies != kRows) return std::printf("%d copies\n", int(g_copies)), 1;
  return 0;
}
