// libnomad: how the callers' float32 arrays may be read.  Their alignment is the caller's (a view may begin anywhere); wide
// loads are used where every row begins on their boundary.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

// rows of d values beginning at `rows` can be read 16 bytes at a time
__host__ __device__ __forceinline__ bool rows_by_16(const float* rows, int32_t d) { return (d & 3) == 0 && ((uintptr_t)rows & 15) == 0; }

// row i of an array of pairs
__device__ __forceinline__ float2 pair_at(const float* __restrict__ pairs, int64_t i) { return make_float2(pairs[2 * i], pairs[2 * i + 1]); }
