// Test infrastructure: the part of the HIP language that csrc/gbmw_pruned.h uses, for a CPU build in
// which one workgroup runs at a time, a fiber per lane (wave.h).  Found before the real header
// because the test puts this folder first on the include path.
#pragma once
#include <math.h>
#include <stdint.h>
#include <string.h>

#define __device__
#define __host__
#define __global__
#define __forceinline__ inline
#define __launch_bounds__(...)
#define __shared__ static                // one workgroup at a time: LDS variables are shared by its fibers

typedef void* hipStream_t;
typedef int hipError_t;
constexpr hipError_t hipSuccess = 0;

struct float2 { float x, y; };
struct float4 { float x, y, z, w; };
struct int2 { int x, y; };
inline float2 make_float2(float x, float y) { return {x, y}; }
inline float4 make_float4(float x, float y, float z, float w) { return {x, y, z, w}; }
inline int2 make_int2(int x, int y) { return {x, y}; }

inline int __float_as_int(float f) { int i; memcpy(&i, &f, 4); return i; }
inline float __int_as_float(int i) { float f; memcpy(&f, &i, 4); return f; }

#include "../wave.h"
