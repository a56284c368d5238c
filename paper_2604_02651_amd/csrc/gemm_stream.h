// What the kernels that stream the rows of tall matrices share.
#pragma once

#include "common.h"

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short i16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));      // gfx950 global loads take any alignment
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned short u16;

#define STREAM_GPTR(p) ((const __attribute__((address_space(1))) void *)(p))
#define STREAM_LPTR(p) ((__attribute__((address_space(3))) void *)(p))
// s_waitcnt vmcnt(n) only (expcnt and lgkmcnt left at their maxima), gfx9 encoding
#define STREAM_WAIT_VMCNT(n) __builtin_amdgcn_s_waitcnt(((n) & 15) | (((n) >> 4) << 14) | 0x0F70)

// ds_read_b64_tr_b16: sixteen lanes read 4 rows x 16 columns and each gets the four values of one column.  __restrict__ says that the
// read is of nothing that a direct load may still be writing (the kernels' own waits see to that); without it the compiler waits for all direct
// loads, the ones just issued among them, in front of such a read, and nothing is in flight behind the slice being multiplied (a layer of
// 2^20 rows, 256 x 256, of which the product of gemm_tn.hip was a fifth: 1288 -> 1257 us; 2^18 rows 517 -> 509).
__device__ __forceinline__ uint2 read_tr(const unsigned char *__restrict__ p)
{
    return __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) i16x4 *)(p)));
}

// v moved down by s places, zeros from above: four values from within the last four of a row, loaded as the four that end with it
__device__ __forceinline__ f32x4 shifted(f32x4 v, int s)
{
    v = (s & 1) ? f32x4{v[1], v[2], v[3], 0.f} : v;
    v = (s & 2) ? f32x4{v[2], v[3], 0.f, 0.f} : v;
    return s >= 4 ? f32x4{0.f, 0.f, 0.f, 0.f} : v;
}

__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi)
{
    return (uint32_t)__builtin_bit_cast(u16, (__bf16)lo) | (uint32_t)__builtin_bit_cast(u16, (__bf16)hi) << 16;
}
