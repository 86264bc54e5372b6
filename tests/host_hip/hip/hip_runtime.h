// What csrc/eco_device.h needs of HIP to be compiled for the CPU: its arithmetic is then
// run by noise_accuracy_check.cpp.  Not used by the library.
#pragma once
#include <cmath>
#include <cstdint>
#include <cstring>

#define __device__
#define __forceinline__ inline __attribute__((always_inline))

struct uint4 { uint32_t x, y, z, w; };
struct float4 { float x, y, z, w; };
struct double2 { double x, y; };
inline uint4 make_uint4(uint32_t x, uint32_t y, uint32_t z, uint32_t w) { return {x, y, z, w}; }
inline double2 make_double2(double x, double y) { return {x, y}; }
inline double __hiloint2double(int hi, int lo) {
  const uint64_t b = (uint64_t)(uint32_t)hi << 32 | (uint32_t)lo;
  double d;
  std::memcpy(&d, &b, 8);
  return d;
}
struct Dim { uint32_t x; };
static const Dim threadIdx{0}, blockDim{1};
inline void __syncthreads() {}

// The hardware's reciprocal square root is within 2^-24 of the value: here off by as much
// as the check asks for.
extern double rsq_off;
inline double __builtin_amdgcn_rsq(double y) { return (double)((1.0L / std::sqrt((long double)y)) * (1.0L + rsq_off)); }
inline uint32_t __builtin_amdgcn_bitop3_b32(uint32_t a, uint32_t b, uint32_t c, uint32_t) { return a ^ b ^ c; }
inline void __builtin_amdgcn_fence(int, const char*) {}
inline void __builtin_amdgcn_wave_barrier() {}
