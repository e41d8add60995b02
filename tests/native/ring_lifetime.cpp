// The upload ring on the host: "device" memory is ordinary memory and a copy takes place when
// it is issued.  Tables are staged in groups, each group partly of tables that are staged
// already, at every fill level of the ring; when a group is launched, all its tables must hold
// what was put.
#include <cstdio>
#include <cstdlib>
#include <random>

#include "driver_util.hpp"

extern "C" {
hipError_t hipHostMalloc(void** p, size_t bytes, unsigned) { return (*p = std::malloc(bytes)) ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipHostFree(void* p) { std::free(p); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t bytes, hipMemcpyKind, hipStream_t) {
  std::memcpy(d, s, bytes);
  return hipSuccess;
}
const char* hipGetErrorString(hipError_t) { return "error"; }
}

namespace sislice {
void* ws_get(sislice_handle*, int, size_t bytes) { return std::calloc(bytes, 1); }
}  // namespace sislice

int main() {
  using namespace sislice;
  sislice_handle h;
  Ring ring(&h, 64 * 256);
  std::mt19937 rng(7);
  int bad = 0;
  for (int group = 0; group < 20000; ++group) {
    // up to 16 tables (a quarter of the ring), most of them from a small pool
    const int count = 1 + (int)(rng() % 16);
    std::vector<std::vector<int>> want;
    std::vector<int*> got;
    for (int t = 0; t < count; ++t) {
      const int id = rng() % 4 ? (int)(rng() % 24) : 1000 + group * 16 + t;
      want.push_back(std::vector<int>(1 + id % 60, id));
      got.push_back(ring.vec(want.back()));
    }
    h.flush_fn(h.flush_ctx);  // the launch
    for (int t = 0; t < count; ++t)
      bad += std::memcmp(got[t], want[t].data(), want[t].size() * sizeof(int)) != 0;
    if (rng() % 50 == 0) ring.synced();
  }
  if (bad) std::printf("%d tables overwritten before their launch\n", bad);
  return bad != 0;
}
