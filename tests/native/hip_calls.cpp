// Stand-ins for the HIP calls of the library's set-up, on the CPU: "device"
// memory is host memory, launches do nothing, and the calls are counted.
// Preloaded, so that the library's calls come here.
#include <cstdlib>
#include <cstring>

#define API extern "C" __attribute__((visibility("default")))

static int copies, queries, launches;
API int calls_of(int what) { return what == 0 ? copies : what == 1 ? queries : launches; }

API int hipGetDevice(int *dev) { return *dev = 0; }
API int hipDeviceGetAttribute(int *v, int, int) { return *v = 256, 0; }
API int hipGetSymbolAddress(void **p, const void *) {
  static void *mem = std::calloc(8 << 20, 1);
  return *p = mem, 0;
}
API int hipMemsetAsync(void *p, int v, size_t n, void *) { return std::memset(p, v, n), 0; }
API int hipMemcpyAsync(void *d, const void *s, size_t n, int, void *) {
  return ++copies, std::memcpy(d, s, n), 0;
}
API int hipStreamSynchronize(void *) { return 0; }
API int hipGetLastError() { return 0; }
API int hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *, int, size_t) {
  return ++queries, *n = 4, 0;
}
struct Dim3 {
  unsigned x, y, z;
};
API int __hipPushCallConfiguration(Dim3, Dim3, size_t, void *) { return 0; }
API int __hipPopCallConfiguration(Dim3 *, Dim3 *, size_t *n, void **s) { return *n = 0, *s = 0, 0; }
API int hipLaunchKernel(const void *, Dim3, Dim3, void **, size_t, void *) {
  return ++launches, 0;
}
