// The residue accumulators of a call on a device whose memory is short: a
// fake allocator with a budget behind Scratch::reserve_acc (common.cpp).
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>

#include "../paper_2106_03058_amd/csrc/agp_internal.h"

static size_t budget, held;
static std::map<void*, size_t> blocks;

extern "C" {
hipError_t hipMalloc(void** p, size_t n) {
  if (held + n > budget) return hipErrorOutOfMemory;
  *p = std::malloc(n);
  blocks[*p] = n;
  held += n;
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  held -= blocks.at(p);
  blocks.erase(p);
  std::free(p);
  return hipSuccess;
}
hipError_t hipMemsetAsync(void* p, int v, size_t n, hipStream_t) {
  std::memset(p, v, n);
  return hipSuccess;
}
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) {
  std::memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipGetLastError(void) { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "fake"; }
hipError_t hipEventCreate(hipEvent_t*) { return hipErrorNotSupported; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
}

static bool zeros(const agp::DevBuf& b, size_t n) {
  for (size_t i = 0; i < n; ++i)
    if (b.as<unsigned char>()[i]) return false;
  return true;
}

// argv: budget, bytes of one copy, bytes that each buffer holds before (0: none)
int main(int argc, char** argv) {
  if (argc != 4) return 2;
  budget = std::strtoull(argv[1], nullptr, 10);
  const size_t bytes = std::strtoull(argv[2], nullptr, 10), before = std::strtoull(argv[3], nullptr, 10);
  agp::Scratch sc;
  if (before)
    for (auto& b : sc.acc)
      if (b.reserve(before, true, nullptr)) return 3;
  int copies = 4;
  const int rc = sc.reserve_acc(bytes, &copies, nullptr);
  if (rc == AGP_OK)
    for (auto& b : sc.acc)
      if (b.bytes < bytes * copies || !zeros(b, bytes * copies)) return 4;
  std::printf("%d %d %zu\n", rc, copies, held);
  sc.release();
  return held == 0 ? 0 : 5;
}
