/* Host stand-ins for the HIP calls of libpt.so, for CPU tests of what the library does when the
 * device has no memory left.  Loaded with RTLD_GLOBAL before libpt.so, so its definitions come
 * first.  Kernels do nothing; "device" memory is untouched host memory, so that large buffers
 * cost nothing, and is counted against a budget the test sets. */
#define _GNU_SOURCE
#include <stddef.h>
#include <stdint.h>
#include <string.h>
#include <sys/mman.h>

enum { kOk = 0, kOutOfMemory = 2 };
static const size_t kTotal = (size_t)1 << 36; /* 64 GiB of address space at most */
static size_t budget = (size_t)1 << 36, held, peak;
static long fail_in, mallocs, launches;
static int last_error;

/* the n-th hipMalloc from now and all after it fail (n >= 1; 0: none) */
void stub_fail_malloc(long n) { fail_in = n; }
void stub_budget(size_t bytes) { budget = bytes; }
size_t stub_held(void) { return held; }
size_t stub_peak(void) { size_t p = peak; peak = held; return p; }
long stub_mallocs(void) { return mallocs; }
long stub_launches(void) { return launches; }

static size_t span(size_t n) { return (n + sizeof(size_t) + 4095) / 4096 * 4096 + 4096; }
int hipMalloc(void** p, size_t n) {
  *p = NULL;
  ++mallocs;
  if (fail_in > 1) --fail_in;
  else if (fail_in == 1) return last_error = kOutOfMemory;
  if (held + n > budget || n > kTotal) return last_error = kOutOfMemory;
  char* m = mmap(NULL, span(n), PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
  if (m == MAP_FAILED) return last_error = kOutOfMemory;
  *(size_t*)m = n;
  held += n;
  if (held > peak) peak = held;
  *p = m + 4096;
  return kOk;
}
int hipFree(void* p) {
  if (!p) return kOk;
  char* m = (char*)p - 4096;
  const size_t n = *(size_t*)m;
  held -= n;
  munmap(m, span(n));
  return kOk;
}
int hipMemGetInfo(size_t* avail, size_t* total) {
  *avail = budget - held;
  *total = kTotal;
  return kOk;
}
int hipHostMalloc(void** p, size_t n, unsigned flags) {
  static char words[1 << 16];
  static size_t used;
  if (used + n > sizeof(words)) return last_error = kOutOfMemory;
  *p = words + used;
  used += (n + 63) & ~(size_t)63;
  return kOk;
}
int hipHostFree(void* p) { return kOk; }
int hipMemcpyAsync(void* dst, const void* src, size_t n, int kind, void* stream) {
  if (kind != 3) memcpy(dst, src, n); /* device to device: what kernels would have written is not there either */
  return kOk;
}
int hipMemsetAsync(void* dst, int v, size_t n, void* stream) { return kOk; }
int hipLaunchKernel(const void* f, uint64_t g0, uint32_t g1, uint64_t b0, uint32_t b1, void** args, size_t lds,
                    void* stream) {
  ++launches;
  return kOk;
}
int hipGetLastError(void) {
  const int e = last_error;
  last_error = kOk;
  return e;
}
int hipGetDeviceCount(int* n) { *n = 1; return kOk; }
int hipGetDevice(int* d) { *d = 0; return kOk; }
int hipSetDevice(int d) { return kOk; }
int hipDeviceGetAttribute(int* v, int attr, int dev) { *v = 256; return kOk; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void* f, int block, size_t lds) { *n = 6; return kOk; }
int hipGetSymbolAddress(void** p, const void* symbol) {
  static char scratch[1 << 20];
  *p = scratch;
  return kOk;
}
static char handle[64];
int hipStreamCreateWithFlags(void** s, unsigned flags) { *s = handle; return kOk; }
int hipStreamDestroy(void* s) { return kOk; }
int hipStreamSynchronize(void* s) { return kOk; }
int hipStreamWaitEvent(void* s, void* e, unsigned flags) { return kOk; }
int hipEventCreate(void** e) { *e = handle; return kOk; }
int hipEventCreateWithFlags(void** e, unsigned flags) { *e = handle; return kOk; }
int hipEventDestroy(void* e) { return kOk; }
int hipEventRecord(void* e, void* s) { return kOk; }
int hipEventSynchronize(void* e) { return kOk; }
int hipEventElapsedTime(float* ms, void* a, void* b) { *ms = 0.0f; return kOk; }
