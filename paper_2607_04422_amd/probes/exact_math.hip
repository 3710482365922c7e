// Sweeps of the device helpers whose results are said to be those of the general operations:
// each counts the values where they differ.  Built into libfp4root_sweeps.so for the tests
// (the kernels of the library use the same helpers from device.h).
#include "../csrc/device.h"

namespace {
using namespace fp4r;

constexpr uint32_t kBlocks = 8192;

// out[0]: number of differences, out[1]: the bits of one value that differs
__device__ void report(uint32_t* out, uint32_t bad, uint32_t which) {
  if (bad == 0) return;
  atomicAdd(&out[0], bad);
  out[1] = which;
}

__global__ __launch_bounds__(256) void k_sqrt(uint32_t first, uint32_t count, uint32_t* out) {
  uint32_t bad = 0, which = 0;
  for (uint64_t i = blockIdx.x * 256u + threadIdx.x; i < count; i += kBlocks * 256u) {
    const uint32_t bits = first + (uint32_t)i;
    const float v = __uint_as_float(bits);
    if (__float_as_uint(fast_sqrt(v)) != __float_as_uint(__builtin_sqrtf(v))) {
      ++bad;
      which = bits;
    }
  }
  report(out, bad, which);
}

__global__ __launch_bounds__(256) void k_bf16(uint32_t first, uint32_t count, uint32_t* out) {
  uint32_t bad = 0, which = 0;
  for (uint64_t i = blockIdx.x * 256u + threadIdx.x; i < count; i += kBlocks * 256u) {
    const uint32_t bits = first + (uint32_t)i;
    const float v = __uint_as_float(bits);
    const uint32_t want = (uint32_t)bf16_rne(v) | ((uint32_t)bf16_rne(-v) << 16);
    if (bf16_pair(v, -v) != want) {
      ++bad;
      which = bits;
    }
  }
  report(out, bad, which);
}

// Quotients a / b by the binary64 reciprocals of the AdamW step: a of either sign in
// [2^-126, 2^127), b in [2^-100, 2^21]; counted where a / b is a normal number or overflows.
__global__ __launch_bounds__(256) void k_div(uint64_t seed, uint32_t count, uint32_t* out) {
  uint32_t bad = 0, which = 0;
  for (uint64_t i = blockIdx.x * 256u + threadIdx.x; i < count; i += kBlocks * 256u) {
    const uint64_t z = splitmix64_at(seed, i + 1);
    const uint32_t ab = 0x00800000u + (uint32_t)(((z >> 32) * 0x7E800000ull) >> 32);
    const uint32_t bb = 0x0D800000u + (uint32_t)(((z & 0xFFFFFFFFull) * (0x4A000000ull - 0x0D800000ull + 1)) >> 32);
    const float a = __uint_as_float(ab | ((uint32_t)(z & 1u) << 31)), b = __uint_as_float(bb);
    const float want = a / b;
    if (!(fabsf(want) >= 0x1p-126f)) continue;
    const uint32_t w = __float_as_uint(want);
    if (__float_as_uint(fast_div(a, 1.0 / (double)b)) != w || __float_as_uint(fast_div(a, recip64(b))) != w) {
      ++bad;
      which = ab;
    }
  }
  report(out, bad, which);
}
}  // namespace

extern "C" {
int fp4root_sweep_sqrt(uint32_t first, uint32_t count, uint32_t* out, void* stream) {
  hipLaunchKernelGGL(k_sqrt, dim3(kBlocks), dim3(256), 0, (hipStream_t)stream, first, count, out);
  return (int)hipGetLastError();
}
int fp4root_sweep_bf16(uint32_t first, uint32_t count, uint32_t* out, void* stream) {
  hipLaunchKernelGGL(k_bf16, dim3(kBlocks), dim3(256), 0, (hipStream_t)stream, first, count, out);
  return (int)hipGetLastError();
}
int fp4root_sweep_div(uint64_t seed, uint32_t count, uint32_t* out, void* stream) {
  hipLaunchKernelGGL(k_div, dim3(kBlocks), dim3(256), 0, (hipStream_t)stream, seed, count, out);
  return (int)hipGetLastError();
}
}
