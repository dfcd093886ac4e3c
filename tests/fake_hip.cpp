// A HIP runtime without a device, for host-side tests of libfwime.so: device
// memory is address space that is counted and never touched, kernels are
// counted by name and not run, except that those whose results the host reads
// (input checks, inner products) are answered with finite values.  Loaded with RTLD_GLOBAL ahead of the library.
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <string>
#include <vector>

namespace {
constexpr int kOutOfMemory = 2, kInvalid = 1;
struct Dim3 { unsigned x, y, z; };
std::recursive_mutex mu;
size_t total = (size_t)288 << 30, other = 0, used = 0, peak = 0, largest_ok = SIZE_MAX;
uintptr_t next_address = (uintptr_t)1 << 44;
std::map<uintptr_t, size_t> live;
std::map<const void *, std::string> names;
std::map<std::string, long> launched;
struct Call { Dim3 grid, block; size_t shmem; void *stream; };
std::vector<Call> calls;
int last = 0;
long allocations = 0;

int fail(int e) { return last = e; }

int allocate(void **p, size_t n) {
  std::lock_guard<std::recursive_mutex> lock(mu);
  *p = nullptr;
  if (n > largest_ok || used + other + n > total) return fail(kOutOfMemory);
  *p = reinterpret_cast<void *>(next_address);
  live[next_address] = n;
  ++allocations;
  next_address += (n + 4095) / 4096 * 4096 + 4096;
  used += n;
  if (used > peak) peak = used;
  return 0;
}

int release(void *p) {
  std::lock_guard<std::recursive_mutex> lock(mu);
  if (!p) return 0;
  auto it = live.find((uintptr_t)p);
  if (it == live.end()) return fail(kInvalid);
  used -= it->second;
  live.erase(it);
  return 0;
}
}  // namespace

extern "C" {
// controls: device size, memory held by others, the largest single allocation that succeeds
void fake_device(size_t bytes, size_t held_by_others) { total = bytes; other = held_by_others; }
void fake_largest(size_t bytes) { largest_ok = bytes; }
size_t fake_used() { return used; }
size_t fake_peak() { return peak; }
void fake_reset() { peak = used; }
long fake_allocations() { return allocations; }
long fake_launched(const char *part) {
  long n = 0;
  for (auto &l : launched)
    if (l.first.find(part) != std::string::npos) n += l.second;
  return n;
}

void **__hipRegisterFatBinary(const void *) {
  static void *handle;
  return &handle;
}
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *, void *, void *, void *,
                           int *) {
  names[host] = name;
}
void __hipRegisterVar(void **, void *, char *, const char *, int, size_t, int, int) {}
int __hipPushCallConfiguration(Dim3 g, Dim3 b, size_t shmem, void *stream) {
  calls.push_back({g, b, shmem, stream});
  return 0;
}
int __hipPopCallConfiguration(Dim3 *g, Dim3 *b, size_t *shmem, void **stream) {
  const Call c = calls.back();
  calls.pop_back();
  *g = c.grid;
  *b = c.block;
  *shmem = c.shmem;
  *stream = c.stream;
  return 0;
}
int hipLaunchKernel(const void *f, Dim3 grid, Dim3, void **args, size_t, void *) {
  const std::string &name = names[f];
  ++launched[name];
  if (name.find("k_ranges") != std::string::npos) {      // (RangeArgs, double *out): min, max, non-finite count
    double *out = *static_cast<double **>(args[1]);
    for (unsigned b = 0; b < grid.x; ++b) {
      out[3 * b] = out[3 * b + 1] = 1500.0;
      out[3 * b + 2] = 0.0;
    }
  }
  if (name.find("k_lbfgs_gram") != std::string::npos) {  // (LbfgsVectors, long n, double *out): partial products
    double *out = *static_cast<double **>(args[2]);
    for (unsigned i = 0; i < grid.x * grid.y * 64; ++i) out[i] = 1.0;
  }
  return 0;
}
int hipMalloc(void **p, size_t n) { return allocate(p, n); }
int hipMallocAsync(void **p, size_t n, void *) { return allocate(p, n); }
int hipFree(void *p) { return release(p); }
int hipFreeAsync(void *p, void *) { return release(p); }
int hipHostMalloc(void **p, size_t n, unsigned) { return (*p = std::calloc(1, n)) ? 0 : fail(kOutOfMemory); }
int hipHostFree(void *p) {
  std::free(p);
  return 0;
}
int hipMemGetInfo(size_t *free_bytes, size_t *total_bytes) {
  *free_bytes = total - other - used;
  *total_bytes = total;
  return 0;
}
int hipMemcpyAsync(void *dst, const void *, size_t n, int kind, void *) {
  if (kind == 2 && n == sizeof(double)) {                 // device to host: an inner product
    const double one = 1.0;
    std::memcpy(dst, &one, sizeof one);
  }
  return 0;
}
int hipGetSymbolAddress(void **p, const void *) {
  *p = reinterpret_cast<void *>((uintptr_t)1 << 43);
  return 0;
}
int hipGetDeviceCount(int *n) {
  *n = 1;
  return 0;
}
int hipSetDevice(int) { return 0; }
int hipDeviceSynchronize() { return 0; }
int hipGetLastError() {
  const int e = last;
  last = 0;
  return e;
}
const char *hipGetErrorString(int) { return "error"; }
int hipStreamSynchronize(void *) { return 0; }
int hipStreamCreateWithFlags(void **s, unsigned) {
  *s = reinterpret_cast<void *>(1);
  return 0;
}
int hipStreamDestroy(void *) { return 0; }
int hipStreamBeginCapture(void *, int) { return 0; }
int hipStreamEndCapture(void *, void **g) {
  *g = reinterpret_cast<void *>(1);
  return 0;
}
int hipGraphInstantiate(void **e, void *, void *, char *, size_t) {
  *e = reinterpret_cast<void *>(1);
  return 0;
}
int hipGraphLaunch(void *, void *) { return 0; }
int hipGraphDestroy(void *) { return 0; }
int hipGraphExecDestroy(void *) { return 0; }
int hipEventCreate(void **e) {
  *e = reinterpret_cast<void *>(1);
  return 0;
}
int hipEventCreateWithFlags(void **e, unsigned) { return hipEventCreate(e); }
int hipEventDestroy(void *) { return 0; }
int hipEventRecord(void *, void *) { return 0; }
int hipEventSynchronize(void *) { return 0; }
int hipEventQuery(void *) { return 0; }
int hipEventElapsedTime(float *ms, void *, void *) {
  *ms = 1.f;
  return 0;
}
}
