// Draw-only loops over the sampling step's own functions: what a draw costs at
// the least.  The counter words may change from step to step, as a lane's do.
#include "../paper_2106_03058_amd/csrc/agp_device.h"

template <bool kSecond, bool kDense>
__device__ __forceinline__ void draws(uint32_t n, const uint32_t* ctr, uint32_t k0, uint32_t k1, const double* p,
                                      uint32_t* out, double* second) {
  const agp::SkipTable t = agp::make_skip_table(p[threadIdx.x]);
  uint32_t a = ctr[threadIdx.x], b = ctr[threadIdx.x + 64], c = ctr[threadIdx.x + 128], d = ctr[threadIdx.x + 192];
  uint32_t skip = 0;
  double v = 0.0;
#pragma unroll 1
  for (uint32_t i = 0; i < n; ++i) {
    __asm__ volatile("" : "+v"(a), "+v"(b), "+v"(c), "+v"(d));
    const agp::U4 o = agp::philox4x32_10_skey(a, b, c, d, k0, k1);
    const double u = agp::unit_double(o.x, o.y);
    skip = kDense ? static_cast<uint32_t>(agp::geometric_skip(t, u)) : agp::geometric_skip64(t, u);
    __asm__ volatile("" : "+v"(skip));
    if (kSecond) {
      v = agp::unit_double(o.z, o.w);
      __asm__ volatile("" : "+v"(v));
    }
  }
  out[threadIdx.x] = skip;
  if (kSecond) second[threadIdx.x] = v;
}

#define LOOP(name, kSecond, kDense)                                                                                  \
  extern "C" __global__ void name(uint32_t n, const uint32_t* c, uint32_t k0, uint32_t k1, const double* p,          \
                                  uint32_t* out, double* second) {                                                   \
    draws<kSecond, kDense>(n, c, k0, k1, p, out, second);                                                            \
  }
LOOP(draws_a0, false, false)
LOOP(draws_ap, true, false)
LOOP(draws_dense, true, true)
