// Exact split of fp32 values into three bfloat16 parts, shared by the kernels that multiply such parts (gemm_split.hip says how and why).
// Included inside their anonymous namespaces.
#pragma once

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
// 16 bytes at any multiple of four (gfx950 global loads take any alignment)
typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));

constexpr uint32_t TINY = 2u * ((127u - 112u) << 23) - 1u;   // tiny_key() of 2^-112

// four values -> their three parts, packed
struct parts4 { uint2 p[3]; };
__device__ __forceinline__ uint32_t cvt2(float a, float b) { return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{a, b}, bf16x2)); }
__device__ __forceinline__ float lo16(uint32_t w) { return __builtin_bit_cast(float, w << 16); }
__device__ __forceinline__ float hi16(uint32_t w) { return __builtin_bit_cast(float, w & 0xffff0000u); }
__device__ __forceinline__ void split2(float x, float y, uint32_t &p1, uint32_t &p2, uint32_t &p3)
{
    p1 = cvt2(x, y);
    x -= lo16(p1); y -= hi16(p1);
    p2 = cvt2(x, y);
    x -= lo16(p2); y -= hi16(p2);
    p3 = cvt2(x, y);
}
// a value's bits without the sign, shifted left, less one: in the order of the magnitudes, but zero is the largest
__device__ __forceinline__ uint32_t tiny_key(float x) { return 2u * __builtin_bit_cast(uint32_t, x) - 1u; }
__device__ __forceinline__ parts4 split4(const float (&v)[4], uint32_t &tiny)
{
    parts4 r;
    split2(v[0], v[1], r.p[0].x, r.p[1].x, r.p[2].x);
    split2(v[2], v[3], r.p[0].y, r.p[1].y, r.p[2].y);
    // smallest key seen: of the values themselves, because a value of up to 2^-134 has a zero for its first part
    asm("v_min3_u32 %0, %0, %1, %2" : "+v"(tiny) : "v"(tiny_key(v[0])), "v"(tiny_key(v[1])));
    asm("v_min3_u32 %0, %0, %1, %2" : "+v"(tiny) : "v"(tiny_key(v[2])), "v"(tiny_key(v[3])));
    return r;
}
