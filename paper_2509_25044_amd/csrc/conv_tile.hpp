// Pieces shared by the tiled convolution kernels (forward, input gradients).
#pragma once
#include <hip/hip_runtime.h>

#include "conv_types.hpp"
#include "internal.hpp"

namespace ffdp {

namespace {

struct TcArgs {
    int N, Di, Hi, Wi, Do, Ho, Wo;
    int Ca, Cb, Nout;
    const unsigned short* xa;
    const unsigned short* xb;
    const float* dy;            // FROMDY: part a is dL/dy act'(y)
    const unsigned short* y;
    float slope;
    const unsigned short* w;    // [Nout][27][Ca + Cb]
    const float* bias;
    int act;
    unsigned short* ybf;
    float* yf;
    int accumulate;
    int na, ng, nfrag;          // groups of part a, all groups, weight fragments of an output tile
    int nx, ny, nz, zlen, nnb, nblocks;
    int buf[2];                 // LDS offsets of the two slice buffers (16-byte units)
};

typedef __bf16 bf4v_a8 __attribute__((ext_vector_type(4), aligned(8)));

// what lanes outside the array or past the last channel load
static __device__ uint4 tc_zero;

// global (not flat) loads, also where the address is chosen between an array and tc_zero
typedef const __attribute__((address_space(1))) unsigned short* gptr;
__device__ __forceinline__ gptr as_global(const void* p) { return (gptr)p; }
__device__ __forceinline__ uint4 ld16(gptr p)
{
    const u32x4_a8 v = *reinterpret_cast<const __attribute__((address_space(1))) u32x4_a8*>(p);
    return make_uint4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ uint2 ld8(gptr p)
{
    const u32x2_a8 v = *reinterpret_cast<const __attribute__((address_space(1))) u32x2_a8*>(p);
    return make_uint2(v.x, v.y);
}

// v, unknown to the optimiser: what is formed from it is formed where it stands and not kept in registers across
// the steps (the accumulators leave none to spare)
__device__ __forceinline__ int opaque(int v)
{
    asm volatile("" : "+v"(v));
    return v;
}

__device__ __forceinline__ bf8v as_bf8(uint4 v) { return __builtin_bit_cast(bf8v, v); }

constexpr int TC_LDS = 160 * 1024;

// Blocks of NT threads that fit a CU: LDS, and registers (waves of 8 rows take
// up to 256, waves of fewer rows up to 128).
inline int tc_resident_blocks(int lds, int NT, int RW)
{
    const int by_lds = TC_LDS / lds, by_regs = (RW >= 8 ? 8 : 16) / (NT / 64);
    return by_lds < by_regs ? by_lds : by_regs > 0 ? by_regs : 1;
}

// Columns, z chunks and blocks of a tile of YT rows x WN channel tiles of which
// `resident` blocks fit a CU.  z chunks: the fewest rounds of resident blocks
// times the slices of a block, its two extra input slices counted as one.
inline hipError_t tc_plan(TcArgs& a, int Do, int Ho, int Wo, int YT, int WN, int resident)
{
    a.nnb = (a.Nout + 16 * WN - 1) / (16 * WN);
    a.nx = (Wo + 15) / 16;
    a.ny = (Ho + YT - 1) / YT;
    const long long cols = (long long)a.N * a.nx * a.ny * a.nnb, slots = 256 * resident;
    long long best = -1;
    for (int nz = 1; nz <= Do && (nz == 1 || cols * nz <= 16384); ++nz) {
        const int zl = (Do + nz - 1) / nz, n = (Do + zl - 1) / zl;
        if (n != nz) continue;
        const long long cost = ((cols * n + slots - 1) / slots) * (zl + 1);
        if (best < 0 || cost < best) { best = cost; a.zlen = zl; a.nz = n; }
        if (cols * (Do + n) >= best * slots) break;  // no later count can be below that / slots
    }
    const long long nb = cols * a.nz;
    if (nb > 0x7fffffffLL) return hipErrorInvalidValue;
    a.nblocks = (int)nb;
    return hipSuccess;
}

}  // namespace

}  // namespace ffdp
