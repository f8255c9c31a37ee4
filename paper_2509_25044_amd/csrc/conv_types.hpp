// bf16 operand types and conversions shared by the convolution kernels.
#pragma once
#include <hip/hip_runtime.h>

namespace ffdp {

typedef short s4v __attribute__((ext_vector_type(4)));
typedef float f4v __attribute__((ext_vector_type(4)));
typedef __bf16 bf8v __attribute__((ext_vector_type(8)));
typedef short s8v __attribute__((ext_vector_type(8)));

__device__ __forceinline__ unsigned short f2bf(float f)
{
    unsigned u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (unsigned short)((u >> 16) | 0x40u);  // quiet NaN
    return (unsigned short)((u + 0x7fffu + ((u >> 16) & 1u)) >> 16);                  // round to nearest even
}
__device__ __forceinline__ float bf2f(unsigned short h) { return __uint_as_float((unsigned)h << 16); }

__device__ __forceinline__ float lrelu_d(unsigned short y, float slope) { return bf2f(y) > 0.0f ? 1.0f : slope; }

// global 16-byte accesses that need only 8- or 4-byte alignment
typedef unsigned u32x4_a8 __attribute__((ext_vector_type(4), aligned(8)));
typedef unsigned u32x2_a8 __attribute__((ext_vector_type(2), aligned(8)));
typedef float f32x4_a4 __attribute__((ext_vector_type(4), aligned(4)));

__device__ __forceinline__ uint4 ld16(const unsigned short* p)
{
    const u32x4_a8 v = *reinterpret_cast<const u32x4_a8*>(p);
    return make_uint4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ uint2 ld8(const unsigned short* p)
{
    const u32x2_a8 v = *reinterpret_cast<const u32x2_a8*>(p);
    return make_uint2(v.x, v.y);
}

// channels c .. c + 7 of the voxel at p, which has C (a multiple of 4) channels; zeros past C
__device__ __forceinline__ uint4 load_c8(const unsigned short* __restrict__ p, int c, int C)
{
    if (c + 8 <= C) return ld16(p + c);
    uint2 h = make_uint2(0u, 0u);
    if (c + 4 <= C) h = ld8(p + c);
    return make_uint4(h.x, h.y, 0u, 0u);
}

__device__ __forceinline__ unsigned p_pack2(float a, float b) { return (unsigned)f2bf(a) | ((unsigned)f2bf(b) << 16); }

// 4 channels of P from dL/dy and y (y NULL: no activation)
__device__ __forceinline__ uint2 p_from_dy4(const float* __restrict__ dy, const unsigned short* __restrict__ y,
                                            float slope, size_t o)
{
    const f32x4_a4 d = *reinterpret_cast<const f32x4_a4*>(dy + o);
    float v[4] = {d.x, d.y, d.z, d.w};
    if (y) {
        const uint2 yv = ld8(y + o);
        const unsigned yw[2] = {yv.x, yv.y};
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] *= lrelu_d((unsigned short)(yw[q >> 1] >> (16 * (q & 1))), slope);
    }
    return make_uint2(p_pack2(v[0], v[1]), p_pack2(v[2], v[3]));
}

// 8 channels c .. c + 7 of P from dL/dy and y at the voxel's element offset o (Cout channels, zeros past them)
__device__ __forceinline__ uint4 p_from_dy8(const float* __restrict__ dy, const unsigned short* __restrict__ y,
                                            float slope, size_t o, int c, int Cout)
{
    uint4 r = make_uint4(0u, 0u, 0u, 0u);
    if (c < Cout) {
        const uint2 h = p_from_dy4(dy, y, slope, o + c);
        r.x = h.x; r.y = h.y;
    }
    if (c + 4 < Cout) {
        const uint2 h = p_from_dy4(dy, y, slope, o + c + 4);
        r.z = h.x; r.w = h.y;
    }
    return r;
}

// The same in two steps, so that the loads can be in flight meanwhile: 8
// channels of dy and y as read (past Cout dy 0 and y 1, so that P is 0 there
// whatever the slope), then P.
struct P8 {
    f32x4_a4 d0 = {0.f, 0.f, 0.f, 0.f}, d1 = {0.f, 0.f, 0.f, 0.f};
    uint2 y0 = make_uint2(0x3f803f80u, 0x3f803f80u), y1 = make_uint2(0x3f803f80u, 0x3f803f80u);
};
__device__ __forceinline__ P8 p8_load(const float* __restrict__ dy, const unsigned short* __restrict__ y, size_t o,
                                      int c, int Cout)
{
    P8 r;
    if (c < Cout) {
        r.d0 = *reinterpret_cast<const f32x4_a4*>(dy + o + c);
        if (y) r.y0 = ld8(y + o + c);
    }
    if (c + 4 < Cout) {
        r.d1 = *reinterpret_cast<const f32x4_a4*>(dy + o + c + 4);
        if (y) r.y1 = ld8(y + o + c + 4);
    }
    return r;
}
__device__ __forceinline__ uint2 p4_form(f32x4_a4 d, uint2 y, bool act, float slope)
{
    float v[4] = {d.x, d.y, d.z, d.w};
    if (act) {
        const unsigned yw[2] = {y.x, y.y};
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] *= lrelu_d((unsigned short)(yw[q >> 1] >> (16 * (q & 1))), slope);
    }
    return make_uint2(p_pack2(v[0], v[1]), p_pack2(v[2], v[3]));
}
__device__ __forceinline__ uint4 p8_form(const P8& r, bool act, float slope)
{
    const uint2 lo = p4_form(r.d0, r.y0, act, slope), hi = p4_form(r.d1, r.y1, act, slope);
    return make_uint4(lo.x, lo.y, hi.x, hi.y);
}

}  // namespace ffdp
