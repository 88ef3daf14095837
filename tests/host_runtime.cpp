// Stand-in for the runtime calls skv_tree.hip makes, linked with it in place of the HIP runtime: device memory is host
// memory, copies are done at once, kernels do nothing.  Counts the calls; pinned memory can be refused, and one of the copies, launches
// and waits to come can fail.
#include <cstddef>
#include <cstdint>
#include <cstdlib>
#include <cstring>

struct Dim {
  uint32_t x, y, z;
};
static long n_calls = 0, n_pinned = 0;
static int refuse_pinned = 0, launched = 0;
static long fail_in = 0;   // the copy, launch or wait that fails, counted from here; 0: none
static int fails() { return ++n_calls, fail_in > 0 && --fail_in == 0; }

extern "C" {
long host_calls() { return n_calls; }
long host_pinned() { return n_pinned; }
void host_refuse_pinned(int on) { refuse_pinned = on; }
void host_fail_in(long calls) { fail_in = calls; }

int hipGetDevice(int* device) {
  ++n_calls;
  *device = 0;
  return 0;
}
int hipMemcpyAsync(void* dst, const void* src, size_t n, int, void*) {
  if (fails()) return 1;
  memcpy(dst, src, n);
  return 0;
}
int hipStreamSynchronize(void*) { return fails(); }
int hipGetLastError() {   // of a launch, or behind memory that was refused
  if (!launched) return ++n_calls, 0;
  launched = 0;
  return fails();
}
int hipHostMalloc(void** p, size_t n, unsigned) {
  ++n_calls;
  *p = refuse_pinned ? nullptr : calloc(1, n);
  n_pinned += *p != nullptr;
  return *p ? 0 : 2;
}
int hipHostFree(void* p) {
  ++n_calls;
  --n_pinned;
  free(p);
  return 0;
}
int hipLaunchKernel(const void*, Dim, Dim, void**, size_t, void*) { return ++n_calls, launched = 1, 0; }
int __hipPushCallConfiguration(Dim, Dim, size_t, void*) { return 0; }
int __hipPopCallConfiguration(Dim* grid, Dim* block, size_t* shared, void** stream) {
  *grid = *block = Dim{1, 1, 1};
  *shared = 0;
  *stream = nullptr;
  return 0;
}
void** __hipRegisterFatBinary(const void*) {
  static void* handle;
  return &handle;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void*, char*, const char*, unsigned, void*, void*, void*, void*, int*) {}
}
