// The library's reciprocals against the division, value by value on the GPU.
#include "rf_device.h"

typedef unsigned long long u64;

namespace {

__device__ __forceinline__ bool same(float a, float b) {
  return __float_as_uint(a) == __float_as_uint(b) || (a != a && b != b);
}
__device__ __forceinline__ bool same(double a, double b) {
  return __double_as_longlong(a) == __double_as_longlong(b) || (a != a && b != b);
}

// Every float, 2^20 threads with 2^12 bit patterns each, neighbours in a
// wavefront.
__global__ __launch_bounds__(256) void check_f32(u64* bad) {
  const uint32_t t = blockIdx.x * 256u + threadIdx.x;
  uint32_t n = 0;
  for (uint32_t r = 0; r < 4096u; ++r) {
    const float x = __uint_as_float((r << 20) | t);
    n += same(rf::rcp_rn(x), 1.0f / x) ? 0u : 1u;
  }
  if (n) atomicAdd(bad, (u64)n);
}

__device__ __forceinline__ u64 mix(u64 z) {  // SplitMix64 (Steele, Lea, Flood 2014)
  z += 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

// 2^32 random doubles of both signs, exponents e0 .. e0 + ne - 1.
__global__ __launch_bounds__(256) void check_f64(int e0, int ne, u64* bad) {
  const u64 t = blockIdx.x * 256ull + threadIdx.x;
  uint32_t n = 0;
  for (u64 r = 0; r < 4096u; ++r) {
    const u64 q = mix(t * 4096u + r);
    const u64 e = (u64)(1023 + e0 + (int)(((q >> 52) & 0x7FFu) % (u64)ne));
    const double x = __longlong_as_double((long long)((q & 0x800FFFFFFFFFFFFFull) | (e << 52)));
    n += same(rf::rcp_f64(x), 1.0 / x) ? 0u : 1u;
  }
  if (n) atomicAdd(bad, (u64)n);
}

__global__ void values_f64(const double* x, double* y, int n) {
  const int i = blockIdx.x * 64 + threadIdx.x;
  if (i < n) y[i] = rf::rcp_f64(x[i]);
}

}  // namespace

// *bad (device, zero before): how many values differ.  Return the HIP error.
extern "C" __attribute__((visibility("default"))) int check_rcp_f32(u64* bad, void* stream) {
  check_f32<<<4096, 256, 0, static_cast<hipStream_t>(stream)>>>(bad);
  return (int)hipGetLastError();
}
extern "C" __attribute__((visibility("default"))) int check_rcp_f64(int e0, int ne, u64* bad, void* stream) {
  if (ne < 1 || e0 < -1022 || e0 + ne > 1024) return (int)hipErrorInvalidValue;
  check_f64<<<4096, 256, 0, static_cast<hipStream_t>(stream)>>>(e0, ne, bad);
  return (int)hipGetLastError();
}
extern "C" __attribute__((visibility("default"))) int rcp_f64_values(const double* x, double* y, int n, void* stream) {
  values_f64<<<(n + 63) / 64, 64, 0, static_cast<hipStream_t>(stream)>>>(x, y, n);
  return (int)hipGetLastError();
}
