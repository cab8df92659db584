// Drives the host side of launch_greedy (k_greedy.hip, compiled for the host
// only) against stand-ins for the runtime calls it makes. The LDS limit of a kernel
// function is state that every host thread shares: whatever the batch, a launch
// has to set the same one, and ask for no more than it.
#include <stdio.h>

#include <map>

#include "jacap_internal.hpp"

namespace {
int failures = 0;
std::map<const void*, int> limit;  // per kernel function: the limit last set
size_t asked = 0;                  // dynamic LDS of the last launch
int launches = 0;
dim3 cfg_grid, cfg_block;
size_t cfg_shared;
hipStream_t cfg_stream;
}  // namespace

#define EXPECT(cond)                                               \
  do {                                                             \
    if (!(cond)) {                                                 \
      fprintf(stderr, "FAILED at line %d: %s\n", __LINE__, #cond); \
      ++failures;                                                  \
    }                                                              \
  } while (0)

extern "C" {
hipError_t hipFuncSetAttribute(const void* f, hipFuncAttribute a, int value) {
  EXPECT(a == hipFuncAttributeMaxDynamicSharedMemorySize);
  const auto it = limit.find(f);
  if (it != limit.end()) EXPECT(it->second == value);
  limit[f] = value;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3, dim3, void**, size_t shared, hipStream_t) {
  ++launches;
  asked = shared;
  const auto it = limit.find(f);
  if (shared > 0) EXPECT(it != limit.end() && (size_t)it->second >= shared);
  return hipSuccess;
}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t s, hipStream_t st) {
  cfg_grid = g; cfg_block = b; cfg_shared = s; cfg_stream = st;
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* s, hipStream_t* st) {
  *g = cfg_grid; *b = cfg_block; *s = cfg_shared; *st = cfg_stream;
  return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
void** __hipRegisterFatBinary(const void*) { static void* m; return &m; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void*, char*, const char*, unsigned int, void*, void*, dim3*, dim3*, int*) {}
}

namespace jacap {
TimedPhase::TimedPhase(hipStream_t stream, int phase, bool) : stream_(stream), phase_(phase) {}
TimedPhase::~TimedPhase() {}
}  // namespace jacap

int main() {
  for (int dtype : {JACAP_DTYPE_FP32, JACAP_DTYPE_BF16})
    for (int d : {64, 128})
      for (int n : {1, 8192, 300, 11000, 4000}) {
        jacap_config c{};
        c.dtype = dtype;
        c.head_dim = d;
        c.budget_k = 16;
        c.ridge = 1.0f;
        jacap::Launch L{};
        L.cfg = &c;
        L.geo.D = d;
        L.geo.U = 8;
        L.geo.V = 1;
        L.geo.maxn = n;
        launches = 0;
        EXPECT(jacap::launch_greedy(L, nullptr, nullptr, nullptr, nullptr) == hipSuccess);
        EXPECT(launches == 2);
        EXPECT(asked > 0);  // these lengths take the LDS kernel
      }
  if (failures) return 1;
  printf("greedy launch ok\n");
  return 0;
}
