// For tests that run the library's index arithmetic and store kernels on the CPU: the HIP names that the headers use, as
// plain C++ (clang; one thread at a time, threadIdx and blockIdx are globals).  Lane exchange, matrix and conversion
// instructions only have to compile here: nothing that a test runs goes through them.
#pragma once
#include <math.h>
#include <stddef.h>
#include <stdint.h>
#include <string.h>

#include <algorithm>

#define __global__
#define __device__
#define __host__
#define __shared__ static
#define __forceinline__ inline
#define __launch_bounds__(...)
#define address_space(n) unused
#define asm
#define volatile(...)

struct alignas(8) uint2 { uint32_t x, y; };
struct alignas(16) uint4 { uint32_t x, y, z, w; };
struct alignas(16) float4 { float x, y, z, w; };
struct dim3 { uint32_t x, y, z; dim3(uint32_t x = 1, uint32_t y = 1, uint32_t z = 1) : x(x), y(y), z(z) {} };
inline uint2 make_uint2(uint32_t x, uint32_t y) { return {x, y}; }
inline uint4 make_uint4(uint32_t x, uint32_t y, uint32_t z, uint32_t w) { return {x, y, z, w}; }
inline float4 make_float4(float x, float y, float z, float w) { return {x, y, z, w}; }
inline float __uint_as_float(uint32_t u) { float f; memcpy(&f, &u, 4); return f; }
inline uint32_t __float_as_uint(float f) { uint32_t u; memcpy(&u, &f, 4); return u; }
inline dim3 threadIdx(0, 0, 0), blockIdx(0, 0, 0), blockDim;
using std::max;
using std::min;

#define __syncthreads()
#define __threadfence_block()
#define __shfl_xor(x, m) (x)
#define __builtin_amdgcn_readfirstlane(x) (x)
#define __builtin_amdgcn_readlane(x, l) (x)
#define __builtin_amdgcn_update_dpp(o, x, ...) (x)
#define __builtin_amdgcn_exp2f(x) exp2f(x)
#define __builtin_amdgcn_perm(a, b, s) (0u)
#define __builtin_amdgcn_fdot2(a, b, c, s) (c)
#define __builtin_amdgcn_fdot2_f32_bf16(a, b, c, s) (c)
#define __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(c, s, h) f16x2{}
#define __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(c, s, h) bf16x2{}
#define __builtin_amdgcn_cvt_pk_fp8_f32(a, b, o, h) (((int)(a) & 255) | ((int)(b) & 255) << 8)
