// Host stand-in for the HIP runtime calls that creating a plan makes: device memory is host memory
// with a budget, beyond which allocations fail.  Loaded with global symbols before the library
// (tests/test_plan_memory_host.py), so that plans can be created without a GPU.
#include <cstdlib>
#include <cstring>
#include <map>

namespace {
std::map<void*, size_t> held;
size_t budget = ~size_t{0}, used = 0;
int last = 0;
}  // namespace

extern "C" {
void device_memory_budget(size_t bytes) { budget = bytes; }
size_t device_memory_used() { return used; }

int hipMalloc(void** p, size_t n) {
  if (used + n > budget) {
    *p = nullptr;
    return last = 2;  // hipErrorOutOfMemory
  }
  *p = std::malloc(n);
  held[*p] = n;
  used += n;
  return 0;
}
int hipFree(void* p) {
  const auto it = held.find(p);
  if (it == held.end()) return p ? 1 : 0;
  used -= it->second;
  held.erase(it);
  std::free(p);
  return 0;
}
int hipMemcpy(void* dst, const void* src, size_t n, int) {
  std::memcpy(dst, src, n);
  return 0;
}
int hipGetDevice(int* d) {
  *d = 0;
  return 0;
}
int hipDeviceSynchronize() { return 0; }
int hipGetLastError() {
  const int e = last;
  last = 0;
  return e;
}
int hipEventCreateWithFlags(void** e, unsigned) {
  *e = std::malloc(1);
  return 0;
}
int hipEventDestroy(void* e) {
  std::free(e);
  return 0;
}
}
