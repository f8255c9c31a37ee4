// BF16 MFMA implicit-GEMM 3x3x3 convolutions (pad 1, stride 1 or 2) for the
// warm-start U-Net, gfx950.  FP32 accumulation.
//
// Activations are channels-last bf16 [N][D][H][W][C].  A convolution input
// may be the channel concatenation of an upsampled coarse tensor xa (nearest
// x2, channels [0, Ca)) and a skip tensor xb (channels [Ca, Ca+Cb)); the
// upsampling and the concatenation happen in the operand gather and are never
// materialised.
//
//   forward      y[o][co] = act(b[co] + sum_{t,ci} X[o*s + t - 1][ci] W[co][t][ci])
//   backward-data dX[i][ci] = sum_{t,co} P[(i + 1 - t)/s][co] W[co][t][ci]
// with P = dL/dy * act'(y) (LeakyReLU: slope where y <= 0), formed in the
// gather and rounded to bf16 as the MFMA operand.
//
// Forward and backward-data: each 64-lane wave owns one 16-row slab of the
// GEMM (a block of four waves 64 rows) and issues gfx950's
// v_mfma_f32_16x16x32_bf16 over 32-wide K steps.  Operand layout of that
// instruction (lane l, element e):
//   A[i][k]: i = l % 16, k = 8 (l / 16) + e (e < 8)   B[k][j]: k = 8 (l / 16) + e, j = l % 16
//   D[i][j]: i = 4 (l / 16) + e (e < 4), j = l % 16
// K is ordered (tap, channel); a lane's 8 K elements are two groups of 4
// consecutive channels (channel counts are multiples of 4), each one 8-byte
// load of 4 bf16 (or 16 bytes of fp32 for the backward-data operand).  The
// weight operand of 128 K columns for every output column of the block is
// staged in LDS once per block and read by all four waves (rows padded by 8
// bf16 so that the 16 rows a wave reads fall in different banks).
#include "device.hpp"
#include "internal.hpp"
#include "conv_p.hpp"
#include "conv_types.hpp"

namespace ffdp {

__device__ __forceinline__ s4v ld4bf(const unsigned short* p)
{
    const uint2 v = *reinterpret_cast<const uint2*>(p);
    s4v r;
    r[0] = (short)(v.x & 0xffffu); r[1] = (short)(v.x >> 16);
    r[2] = (short)(v.y & 0xffffu); r[3] = (short)(v.y >> 16);
    return r;
}

__device__ __forceinline__ s4v pack4(float a, float b, float c, float d)
{
    s4v r;
    r[0] = (short)f2bf(a); r[1] = (short)f2bf(b); r[2] = (short)f2bf(c); r[3] = (short)f2bf(d);
    return r;
}

// eight bf16 (bit patterns in shorts) as the MFMA operand type
__device__ __forceinline__ bf8v cat8(s4v lo, s4v hi)
{
    const s8v r = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(bf8v, r);
}

struct Vox {
    int n, z, y, x;
};
__device__ __forceinline__ Vox vox_of(long long o, int D, int H, int W)
{
    Vox v;
    v.x = (int)(o % W); o /= W;
    v.y = (int)(o % H); o /= H;
    v.z = (int)(o % D);
    v.n = (int)(o / D);
    return v;
}

constexpr int CONV_KC = 128;            // K columns of the weight tile staged per round
constexpr int CONV_KCP = CONV_KC + 8;   // LDS row pitch (bf16)

// Stage rows [0, 16 NT) x columns [k0, k0 + KC) of a row-major bf16 weight
// matrix wsrc [rows][K] into LDS (zeros outside rows < nrows, k < K).  Rows
// start 8-byte aligned (K is a multiple of 4), so each thread moves 4 bf16
// per load.
template <int NT>
__device__ __forceinline__ void stage_weights(unsigned short* __restrict__ ws, const unsigned short* __restrict__ wsrc,
                                              int nrows, int K, int k0)
{
    constexpr int Q = NT * 16 * (CONV_KC / 4);  // 4-element groups
    for (int q = threadIdx.x; q < Q; q += 256) {
        const int r = q / (CONV_KC / 4), c = (q - r * (CONV_KC / 4)) * 4;
        uint2 v = make_uint2(0u, 0u);
        if (r < nrows && k0 + c < K) v = *reinterpret_cast<const uint2*>(wsrc + (size_t)r * K + k0 + c);
        *reinterpret_cast<uint2*>(ws + r * CONV_KCP + c) = v;
    }
}

// B operand of one K step from the staged tile: column j of tile jt, K rows
// kk + 8 (l / 16) .. + 8
__device__ __forceinline__ bf8v b_from_lds(const unsigned short* __restrict__ ws, int jt, int lane, int kk)
{
    const uint4 v = *reinterpret_cast<const uint4*>(ws + (jt * 16 + (lane & 15)) * CONV_KCP + kk + (lane >> 4) * 8);
    return __builtin_bit_cast(bf8v, v);
}

// ---------------------------------------------------------------- forward --
// C8: Ca and Cb are multiples of 8, so a lane's 8 K elements are 8
// contiguous channels of one tap and one 16-byte load.  MT: output tiles of
// 16 voxels per wave; each B operand read from LDS feeds MT MFMAs (with one
// voxel tile per wave the LDS reads of the weights, one per MFMA, bound the
// kernel).
template <int NT, bool C8, int MT>
__global__ void __launch_bounds__(256) conv_fwd_kernel(ConvGeom g, const unsigned short* __restrict__ xa,
                                                       const unsigned short* __restrict__ xb,
                                                       const unsigned short* __restrict__ w,
                                                       const float* __restrict__ bias, int act, float slope,
                                                       unsigned short* __restrict__ ybf, float* __restrict__ yf)
{
    __shared__ __attribute__((aligned(16))) unsigned short ws[NT * 16 * CONV_KCP];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int Cin = g.Ca + g.Cb;
    const int K = 27 * Cin;
    const long long M = (long long)g.N * g.Do * g.Ho * g.Wo;
    const long long mb = ((long long)blockIdx.x * 4 + wave) * 16 * MT;  // the wave's first output voxel
    int n[MT], zs[MT], ys[MT], xs[MT];  // each row's input corner (tap 0, 0, 0)
    bool mvalid[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        const long long m = mb + 16 * mt + (lane & 15);
        mvalid[mt] = m < M;
        n[mt] = 0; zs[mt] = 0; ys[mt] = 0; xs[mt] = 0;
        if (mvalid[mt]) {
            const Vox v = vox_of(m, g.Do, g.Ho, g.Wo);
            n[mt] = v.n;
            zs[mt] = v.z * g.stride - 1; ys[mt] = v.y * g.stride - 1; xs[mt] = v.x * g.stride - 1;
        }
    }
    const int Da = g.Di >> 1, Ha = g.Hi >> 1, Wa = g.Wi >> 1;
    auto load_a4 = [&](int mt, int t, int c) {  // channels c..c+3 of tap t (32-bit voxel indices)
        s4v a = s4v{0, 0, 0, 0};
        const int dz = t / 9, dy = (t - 9 * dz) / 3, dx = t - 9 * dz - 3 * dy;
        const int zi = zs[mt] + dz, yi = ys[mt] + dy, xi = xs[mt] + dx;
        if (mvalid[mt] && t < 27 && (unsigned)zi < (unsigned)g.Di && (unsigned)yi < (unsigned)g.Hi &&
            (unsigned)xi < (unsigned)g.Wi) {
            if (c < g.Ca) {
                const unsigned v = g.ups ? ((unsigned)(n[mt] * Da + (zi >> 1)) * Ha + (yi >> 1)) * Wa + (xi >> 1)
                                         : ((unsigned)(n[mt] * g.Di + zi) * g.Hi + yi) * g.Wi + xi;
                a = ld4bf(xa + (size_t)v * g.Ca + c);
            } else {
                const unsigned v = ((unsigned)(n[mt] * g.Di + zi) * g.Hi + yi) * g.Wi + xi;
                a = ld4bf(xb + (size_t)v * g.Cb + (c - g.Ca));
            }
        }
        return a;
    };
    auto load_a8 = [&](int mt, int t, int c) {  // channels c..c+7 of tap t (C8)
        uint4 a = make_uint4(0u, 0u, 0u, 0u);
        const int dz = t / 9, dy = (t - 9 * dz) / 3, dx = t - 9 * dz - 3 * dy;
        const int zi = zs[mt] + dz, yi = ys[mt] + dy, xi = xs[mt] + dx;
        if (mvalid[mt] && t < 27 && (unsigned)zi < (unsigned)g.Di && (unsigned)yi < (unsigned)g.Hi &&
            (unsigned)xi < (unsigned)g.Wi) {
            if (c < g.Ca) {
                const unsigned v = g.ups ? ((unsigned)(n[mt] * Da + (zi >> 1)) * Ha + (yi >> 1)) * Wa + (xi >> 1)
                                         : ((unsigned)(n[mt] * g.Di + zi) * g.Hi + yi) * g.Wi + xi;
                a = *reinterpret_cast<const uint4*>(xa + (size_t)v * g.Ca + c);
            } else {
                const unsigned v = ((unsigned)(n[mt] * g.Di + zi) * g.Hi + yi) * g.Wi + xi;
                a = *reinterpret_cast<const uint4*>(xb + (size_t)v * g.Cb + (c - g.Ca));
            }
        }
        return __builtin_bit_cast(bf8v, a);
    };
    const int kg = (lane >> 4) * 8;
    // the lane's K index k = (tap t, channel c), advanced by 32 per step
    int t = kg / Cin, c = kg - t * Cin;
    f4v acc[MT][NT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[mt][j] = f4v{0.f, 0.f, 0.f, 0.f};
    for (int k0 = 0; k0 < K; k0 += CONV_KC) {
        __syncthreads();
        stage_weights<NT>(ws, w, g.Cout, K, k0);
        __syncthreads();
#pragma unroll
        for (int kk = 0; kk < CONV_KC; kk += 32) {
            if (k0 + kk >= K) break;  // uniform: no all-zero K steps in the last round
            bf8v a[MT];
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                if (C8) {
                    a[mt] = load_a8(mt, t, c);
                } else {
                    const bool wrap = c + 4 >= Cin;  // channels c + 4 .. c + 7 start the next tap (Cin % 4 == 0)
                    a[mt] = cat8(load_a4(mt, t, c), load_a4(mt, wrap ? t + 1 : t, wrap ? c + 4 - Cin : c + 4));
                }
            }
#pragma unroll
            for (int j = 0; j < NT; ++j) {
                const bf8v b = b_from_lds(ws, j, lane, kk);
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
                    acc[mt][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[mt], b, acc[mt][j], 0, 0, 0);
            }
            c += 32;
            while (c >= Cin) { c -= Cin; ++t; }
        }
    }
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int j = 0; j < NT; ++j) {
            const int co = j * 16 + (lane & 15);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const long long mo = mb + 16 * mt + (lane >> 4) * 4 + e;
                if (mo < M && co < g.Cout) {
                    float v = acc[mt][j][e] + (bias ? bias[co] : 0.0f);
                    if (act) v = v > 0.0f ? v : v * slope;
                    if (ybf) ybf[mo * g.Cout + co] = f2bf(v);
                    if (yf) yf[mo * g.Cout + co] = v;
                }
            }
        }
}

// ----------------------------------------------------------- backward data --
// dX over the virtual (concatenated, fine-resolution) input, fp32 [N][Di][Hi][Wi][Cin];
// accumulate = 1 adds to dX.  wt is the weight in [Cin][27][Cout] order.
// C8: Cout is a multiple of 8, so a lane's 8 K elements are 8 contiguous
// output channels of one tap (two 16-byte loads of dL/dy, one of y).
// PAR (stride 2): an input voxel i receives tap d along an axis only where
// i + 1 - d is even (d = 1 for even i, d = 0 or 2 for odd i), so the input
// voxels are split into the 8 parity classes of (z, y, x) and a block takes
// 64 voxels of one class: its K runs over that class's 1 to 8 taps instead
// of all 27 (3.375 on average), and no product is a structural zero.
// PB: P = dL/dy act'(y) arrives precomputed as bf16 in dL/dy's layout (pb),
// so a lane's 8 K elements are one 16-byte load (4 channels: 8 bytes) and no
// conversion; dy and y are not read.
template <int NT, bool C8, bool PAR, bool PB, int MT>
__global__ void __launch_bounds__(256) conv_bwd_data_kernel(ConvGeom g, const float* __restrict__ dy,
                                                            const unsigned short* __restrict__ y, float slope,
                                                            const unsigned short* __restrict__ pb,
                                                            const unsigned short* __restrict__ wt,
                                                            float* __restrict__ dx, int accumulate)
{
    __shared__ __attribute__((aligned(16))) unsigned short ws[NT * 16 * CONV_KCP];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int Cin = g.Ca + g.Cb;
    const long long M = (long long)g.N * g.Di * g.Hi * g.Wi;
    // parity class (PAR): bits 2, 1, 0 = z, y, x parity; rows index the class's
    // voxels over the half-resolution grid Dc x Hc x Wc (rounded up)
    const int Dc = (g.Di + 1) >> 1, Hc = (g.Hi + 1) >> 1, Wc = (g.Wi + 1) >> 1;
    const long long Mc = (long long)g.N * Dc * Hc * Wc;
    const int bpc = PAR ? (int)((Mc + 64 * MT - 1) / (64 * MT)) : 0;  // blocks per class
    const int cls = PAR ? (int)blockIdx.x / bpc : 0;
    const int pz = (cls >> 2) & 1, py = (cls >> 1) & 1, px = cls & 1;
    const int ny = PAR ? 1 + py : 3, nx = PAR ? 1 + px : 3;  // taps per axis
    const int ntap = PAR ? (1 + pz) * ny * nx : 27;
    const int K = ntap * g.Cout;
    // the wave's MT tiles of 16 rows
    const long long m0 = ((long long)(PAR ? (int)blockIdx.x - cls * bpc : (int)blockIdx.x) * 4 + wave) * 16 * MT;
    auto voxel = [&](long long r, int& n_, int& z_, int& y_, int& x_) -> bool {  // row -> voxel
        if (!PAR) {
            if (r >= M) return false;
            const Vox v = vox_of(r, g.Di, g.Hi, g.Wi);
            n_ = v.n; z_ = v.z; y_ = v.y; x_ = v.x;
            return true;
        }
        if (r >= Mc) return false;
        const Vox v = vox_of(r, Dc, Hc, Wc);
        n_ = v.n; z_ = 2 * v.z + pz; y_ = 2 * v.y + py; x_ = 2 * v.x + px;
        return z_ < g.Di && y_ < g.Hi && x_ < g.Wi;
    };
    int n[MT], zi[MT], yi[MT], xi[MT];
    bool mvalid[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        n[mt] = 0; zi[mt] = 0; yi[mt] = 0; xi[mt] = 0;
        mvalid[mt] = voxel(m0 + 16 * mt + (lane & 15), n[mt], zi[mt], yi[mt], xi[mt]);
    }
    // tap number of the class's j-th tap (PAR), else j itself
    auto tap_of = [&](int j) -> int {
        if (!PAR) return j;
        const int jz = j / (ny * nx), jr = j - jz * ny * nx, jy = jr / nx, jx = jr - jy * nx;
        const int dz = pz ? 2 * jz : 1, dyy = py ? 2 * jy : 1, dx_ = px ? 2 * jx : 1;
        return dz * 9 + dyy * 3 + dx_;
    };
    // element offset of P at output channel co of tap t, or -1 where the tap
    // reaches no output voxel (a non-integer or out-of-range output index)
    auto p_offset = [&](int mt, int j, int co) -> long long {  // j: tap index within the class (PAR) or tap
        if (!mvalid[mt] || j >= ntap) return -1;
        const int t = tap_of(j);
        const int dz = t / 9, dyy = (t - 9 * dz) / 3, dx_ = t - 9 * dz - 3 * dyy;
        int oz = zi[mt] + 1 - dz, oy = yi[mt] + 1 - dyy, ox = xi[mt] + 1 - dx_;
        bool ok = oz >= 0 && oy >= 0 && ox >= 0;
        if (g.stride == 2) {
            ok = ok && !(oz & 1) && !(oy & 1) && !(ox & 1);
            oz >>= 1; oy >>= 1; ox >>= 1;
        }
        ok = ok && oz < g.Do && oy < g.Ho && ox < g.Wo;
        return ok ? (long long)(((unsigned)(n[mt] * g.Do + oz) * g.Ho + oy) * g.Wo + ox) * g.Cout + co : -1;
    };
    auto load_p4 = [&](int mt, int t, int co) {  // P = dL/dy * act'(y) at output channels co..co+3 of tap t
        s4v a = s4v{0, 0, 0, 0};
        const long long o = p_offset(mt, t, co);
        if (PB) {
            if (o >= 0) a = ld4bf(pb + o);
        } else if (o >= 0) {
            const float4 d4 = *reinterpret_cast<const float4*>(dy + o);
            float f[4] = {1.f, 1.f, 1.f, 1.f};
            if (y) {
                const s4v yv = ld4bf(y + o);
#pragma unroll
                for (int q = 0; q < 4; ++q) f[q] = lrelu_d((unsigned short)yv[q], slope);
            }
            a = pack4(d4.x * f[0], d4.y * f[1], d4.z * f[2], d4.w * f[3]);
        }
        return a;
    };
    auto load_p8 = [&](int mt, int t, int co) {  // channels co..co+7 of tap t (C8)
        s4v lo = s4v{0, 0, 0, 0}, hi = s4v{0, 0, 0, 0};
        const long long o = p_offset(mt, t, co);
        if (PB) {
            uint4 v = make_uint4(0u, 0u, 0u, 0u);
            if (o >= 0) v = *reinterpret_cast<const uint4*>(pb + o);
            return __builtin_bit_cast(bf8v, v);
        }
        if (o >= 0) {
            const float4 d0 = *reinterpret_cast<const float4*>(dy + o);
            const float4 d1 = *reinterpret_cast<const float4*>(dy + o + 4);
            float f[8] = {1.f, 1.f, 1.f, 1.f, 1.f, 1.f, 1.f, 1.f};
            if (y) {
                const uint4 yv = *reinterpret_cast<const uint4*>(y + o);
                const unsigned yw[4] = {yv.x, yv.y, yv.z, yv.w};
#pragma unroll
                for (int q = 0; q < 8; ++q) f[q] = lrelu_d((unsigned short)(yw[q >> 1] >> (16 * (q & 1))), slope);
            }
            lo = pack4(d0.x * f[0], d0.y * f[1], d0.z * f[2], d0.w * f[3]);
            hi = pack4(d1.x * f[4], d1.y * f[5], d1.z * f[6], d1.w * f[7]);
        }
        return cat8(lo, hi);
    };
    const int kg = (lane >> 4) * 8;
    // the lane's K index k = (tap t, output channel c), advanced by 32 per step
    int t = kg / g.Cout, c = kg - t * g.Cout;
    f4v acc[MT][NT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[mt][j] = f4v{0.f, 0.f, 0.f, 0.f};
    for (int k0 = 0; k0 < K; k0 += CONV_KC) {
        __syncthreads();
        if (PAR) {
            // the class's K columns (j, c) from wt [Cin][27][Cout]: groups of 4
            // channels of one tap (Cout % 4 == 0) are contiguous there
            constexpr int Q = NT * 16 * (CONV_KC / 4);
            const int K27 = 27 * g.Cout;
            for (int q = threadIdx.x; q < Q; q += 256) {
                const int r = q / (CONV_KC / 4), cc = (q - r * (CONV_KC / 4)) * 4;
                uint2 v = make_uint2(0u, 0u);
                const int k = k0 + cc;
                if (r < Cin && k < K) {
                    const int j = k / g.Cout, c4 = k - j * g.Cout;
                    v = *reinterpret_cast<const uint2*>(wt + (size_t)r * K27 + tap_of(j) * g.Cout + c4);
                }
                *reinterpret_cast<uint2*>(ws + r * CONV_KCP + cc) = v;
            }
        } else {
            stage_weights<NT>(ws, wt, Cin, K, k0);
        }
        __syncthreads();
#pragma unroll
        for (int kk = 0; kk < CONV_KC; kk += 32) {
            if (k0 + kk >= K) break;  // uniform: past the last K column
            bf8v a[MT];
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                if (C8) {
                    a[mt] = load_p8(mt, t, c);
                } else {
                    const bool wrap = c + 4 >= g.Cout;  // Cout % 4 == 0
                    a[mt] = cat8(load_p4(mt, t, c), load_p4(mt, wrap ? t + 1 : t, wrap ? c + 4 - g.Cout : c + 4));
                }
            }
#pragma unroll
            for (int j = 0; j < NT; ++j) {
                const bf8v b = b_from_lds(ws, j, lane, kk);
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
                    acc[mt][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[mt], b, acc[mt][j], 0, 0, 0);
            }
            c += 32;
            while (c >= g.Cout) { c -= g.Cout; ++t; }
        }
    }
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        long long vo[4];  // voxels of the lane's 4 output rows of tile mt (-1: none)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            int n_, z_, y_, x_;
            const long long r = m0 + 16 * mt + (lane >> 4) * 4 + e;
            vo[e] = -1;
            if (voxel(r, n_, z_, y_, x_)) vo[e] = PAR ? (((long long)n_ * g.Di + z_) * g.Hi + y_) * g.Wi + x_ : r;
        }
#pragma unroll
        for (int j = 0; j < NT; ++j) {
            const int ci = j * 16 + (lane & 15);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if (vo[e] >= 0 && ci < Cin) {
                    float* p = dx + vo[e] * Cin + ci;
                    *p = accumulate ? *p + acc[mt][j][e] : acc[mt][j][e];
                }
            }
        }
    }
}

// ------------------------------------------------------------ small kernels --
__global__ void __launch_bounds__(256) cast_bf16_kernel(const float* __restrict__ x, long long n,
                                                        unsigned short* __restrict__ y)
{
    for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < n; i += (long long)gridDim.x * 256)
        y[i] = f2bf(x[i]);
}

// W [Cout][27][Cin] fp32 -> bf16 copy and bf16 transpose [Cin][27][Cout]
__global__ void __launch_bounds__(256) weight_prep_kernel(const float* __restrict__ w, int Cout, int Cin,
                                                          unsigned short* __restrict__ wbf,
                                                          unsigned short* __restrict__ wt)
{
    const int n = Cout * 27 * Cin;
    for (int i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256) {
        const int co = i / (27 * Cin), r = i - co * 27 * Cin, t = r / Cin, ci = r - t * Cin;
        const unsigned short h = f2bf(w[i]);
        if (wbf) wbf[i] = h;
        if (wt) wt[((size_t)ci * 27 + t) * Cout + co] = h;
    }
}

// (F, M) fp32 [N][D][H][W] each -> bf16 [N][D][H][W][4] = (F, M, 0, 0)
__global__ void __launch_bounds__(256) pack_pair_kernel(const float* __restrict__ F, const float* __restrict__ M,
                                                        long long nvox, unsigned short* __restrict__ x)
{
    for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < nvox; i += (long long)gridDim.x * 256) {
        uint2 v;
        v.x = (unsigned)f2bf(F[i]) | ((unsigned)f2bf(M[i]) << 16);
        v.y = 0u;
        *reinterpret_cast<uint2*>(x + 4 * i) = v;
    }
}

// split the gradient of a concatenated, upsampled input: dXcat fp32 [N][Di][Hi][Wi][Ca+Cb]
//   dxb[n,z,y,x,c]  (+)= dXcat[..., Ca + c]
//   dxa[n,Z,Y,X,c]  (+)= sum over the 8 fine voxels (2Z+a, 2Y+b, 2X+c) of dXcat[..., c]
// One block per coarse row (n, Z, Y): it writes dxa of that row and dxb of the
// 4 fine rows (2Z + a, 2Y + b) beneath it, so that the two parts of each
// fine voxel's channels are read by the same block at about the same time
// (a cache line holds both).  Work item (X, k): k < Ca/4 sums channel group k
// of the 8 fine voxels of coarse voxel X (in (a, b, c) order); k = Ca/4 +
// 8 f + q copies channel group q of the skip part of fine voxel f = 4a + 2b + c.
// 16-byte loads and stores (Ca and Cb are multiples of 4, the pointers
// 16-byte aligned).
__global__ void __launch_bounds__(256) split_grad_kernel(ConvGeom g, const float* __restrict__ dxc,
                                                         float* __restrict__ dxa, float* __restrict__ dxb, int acc_a,
                                                         int acc_b)
{
    const int Cin = g.Ca + g.Cb;
    const int R = (int)blockIdx.x;
    const int Da = g.Di >> 1, Ha = g.Hi >> 1, Wa = g.Wi >> 1;
    const int Y = R % Ha, Z = (R / Ha) % Da, n = R / (Ha * Da);
    const int Ga = g.Ca >> 2, Gb = g.Cb >> 2, K = Ga + 8 * Gb;
    const int XC = max(1, (1 << 24) / K);  // X positions per pass: 32-bit item indices
    for (int X0 = 0; X0 < Wa; X0 += XC) {
        const int nit = min(XC, Wa - X0) * K;
        for (int it = (int)threadIdx.x; it < nit; it += 256) {
            const int X = X0 + it / K, k = it % K;
            if (k < Ga) {
                float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
                for (int a = 0; a < 2; ++a)
                    for (int b = 0; b < 2; ++b)
                        for (int c = 0; c < 2; ++c) {
                            const size_t f = (((size_t)n * g.Di + 2 * Z + a) * g.Hi + 2 * Y + b) * g.Wi + 2 * X + c;
                            const float4 v = *reinterpret_cast<const float4*>(dxc + f * Cin + 4 * k);
                            s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
                        }
                float4* d = reinterpret_cast<float4*>(dxa + ((size_t)R * Wa + X) * g.Ca + 4 * k);
                if (acc_a) {
                    const float4 o = *d;
                    s = make_float4(o.x + s.x, o.y + s.y, o.z + s.z, o.w + s.w);
                }
                *d = s;
            } else {
                const int kk = k - Ga, fv = kk / Gb, q = kk - fv * Gb;
                const int a = fv >> 2, b = (fv >> 1) & 1, c = fv & 1;
                const size_t f = (((size_t)n * g.Di + 2 * Z + a) * g.Hi + 2 * Y + b) * g.Wi + 2 * X + c;
                const float4 s = *reinterpret_cast<const float4*>(dxc + f * Cin + g.Ca + 4 * q);
                float4* d = reinterpret_cast<float4*>(dxb + f * g.Cb + 4 * q);
                if (acc_b) {
                    const float4 o = *d;
                    *d = make_float4(o.x + s.x, o.y + s.y, o.z + s.z, o.w + s.w);
                } else {
                    *d = s;
                }
            }
        }
    }
}

// MSE between pred [N][D][H][W][Cp] channels 0..2 and target [N][3][D][H][W]:
// grad (written to dpred, channels >= 3 zeroed) and per-block partial sums.
__global__ void __launch_bounds__(256) mse_kernel(const float* __restrict__ pred, int Cp,
                                                  const float* __restrict__ tgt, long long nvox_per, int N,
                                                  float* __restrict__ dpred, double* __restrict__ part, double scale)
{
    __shared__ double red[256];
    double s = 0.0;
    const long long nv = nvox_per * N;
    for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < nv; i += (long long)gridDim.x * 256) {
        const long long n = i / nvox_per, v = i - n * nvox_per;
        for (int c = 0; c < Cp; ++c) {
            float g = 0.f;
            if (c < 3) {
                const float d = pred[i * Cp + c] - tgt[(n * 3 + c) * nvox_per + v];
                s += (double)d * d;
                g = (float)(2.0 * scale) * d;
            }
            if (dpred) dpred[i * Cp + c] = g;
        }
    }
    s = block_sum<256>(s, red);
    if (threadIdx.x == 0) part[blockIdx.x] = s * scale;
}

// *out = sum of the partials (fixed order)
__global__ void __launch_bounds__(256) sum_partials_kernel(const double* __restrict__ part, int n, float* out)
{
    __shared__ double red[256];
    double s = 0.0;
    for (int i = threadIdx.x; i < n; i += 256) s += part[i];
    s = block_sum<256>(s, red);
    if (threadIdx.x == 0) *out = (float)s;
}

// pred [N][D][H][W][Cp] -> displacement [N][3][D][H][W]
__global__ void __launch_bounds__(256) unpack_disp_kernel(const float* __restrict__ pred, int Cp, long long nvox_per,
                                                          int N, float* __restrict__ u)
{
    const long long nv = nvox_per * N;
    for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < nv; i += (long long)gridDim.x * 256) {
        const long long n = i / nvox_per, v = i - n * nvox_per;
        for (int c = 0; c < 3; ++c) u[(n * 3 + c) * nvox_per + v] = pred[i * Cp + c];
    }
}

// ------------------------------------------------------------------ host ----
static unsigned grid_for(long long n, int per = 256, long long cap = 16384)
{
    long long b = (n + per - 1) / per;
    if (b > cap) b = cap;
    if (b < 1) b = 1;
    return (unsigned)b;
}

template <bool C8>
static void launch_fwd(int nt, unsigned blocks, hipStream_t st, const ConvGeom& g, const unsigned short* xa,
                       const unsigned short* xb, const unsigned short* w, const float* bias, int act, float slope,
                       unsigned short* ybf, float* yf)
{
    // up to 2 output-channel tiles: 2 voxel tiles per wave (a block covers 128
    // voxels); with 4 or 8 the kernel is faster with one (fewer registers)
    const unsigned b2 = (blocks + 1) / 2;
    if (nt <= 1) hipLaunchKernelGGL((conv_fwd_kernel<1, C8, 2>), dim3(b2), dim3(256), 0, st, g, xa, xb, w, bias, act, slope, ybf, yf);
    else if (nt <= 2) hipLaunchKernelGGL((conv_fwd_kernel<2, C8, 2>), dim3(b2), dim3(256), 0, st, g, xa, xb, w, bias, act, slope, ybf, yf);
    else if (nt <= 4) hipLaunchKernelGGL((conv_fwd_kernel<4, C8, 1>), dim3(blocks), dim3(256), 0, st, g, xa, xb, w, bias, act, slope, ybf, yf);
    else hipLaunchKernelGGL((conv_fwd_kernel<8, C8, 1>), dim3(blocks), dim3(256), 0, st, g, xa, xb, w, bias, act, slope, ybf, yf);
}

hipError_t conv_fwd_launch(const ConvGeom& g, const unsigned short* xa, const unsigned short* xb,
                           const unsigned short* w, const float* bias, int act, float slope, unsigned short* ybf,
                           float* yf, hipStream_t st)
{
    const long long M = (long long)g.N * g.Do * g.Ho * g.Wo;
    const unsigned blocks = (unsigned)((M + 63) / 64);
    const int nt = (g.Cout + 15) / 16;
    if (nt > 8) return hipErrorInvalidValue;
    if (g.Ca % 8 == 0 && g.Cb % 8 == 0) launch_fwd<true>(nt, blocks, st, g, xa, xb, w, bias, act, slope, ybf, yf);
    else launch_fwd<false>(nt, blocks, st, g, xa, xb, w, bias, act, slope, ybf, yf);
    return hipGetLastError();
}

template <bool C8, bool PAR, bool PB, int MT>
static void launch_bwd_data(int nt, unsigned blocks, hipStream_t st, const ConvGeom& g, const float* dy,
                            const unsigned short* y, float slope, const unsigned short* pb, const unsigned short* wt,
                            float* dx, int accumulate)
{
#define BWD_DATA(T) \
    hipLaunchKernelGGL((conv_bwd_data_kernel<T, C8, PAR, PB, MT>), dim3(blocks), dim3(256), 0, st, g, dy, y, slope, pb, wt, dx, accumulate)
    if constexpr (MT == 2) {  // nt <= 3
        if (nt <= 1) BWD_DATA(1);
        else if (nt <= 2) BWD_DATA(2);
        else BWD_DATA(3);
    } else {  // nt >= 4
        if (nt <= 4) BWD_DATA(4);
        else if (nt <= 6) BWD_DATA(6);
        else if (nt <= 8) BWD_DATA(8);
        else BWD_DATA(12);
    }
#undef BWD_DATA
}

template <bool PB>
static hipError_t bwd_data_dispatch(const ConvGeom& g, const float* dy, const unsigned short* y, float slope,
                                    const unsigned short* pb, const unsigned short* wt, float* dx, int accumulate,
                                    hipStream_t st)
{
    const int nt = (g.Ca + g.Cb + 15) / 16;
    if (nt > 12) return hipErrorInvalidValue;
    // up to 3 input-channel tiles: 2 voxel tiles per wave, so that each LDS
    // read of the weights feeds two MFMAs (a block covers 128 voxels)
    const int MTv = nt <= 3 ? 2 : 1;
    if (g.stride == 2) {  // 8 parity classes of the half-resolution grid (rounded up)
        const long long Mc = (long long)g.N * ((g.Di + 1) / 2) * ((g.Hi + 1) / 2) * ((g.Wi + 1) / 2);
        const unsigned blocks = (unsigned)(8 * ((Mc + 64 * MTv - 1) / (64 * MTv)));
        if (MTv == 2) {
            if (g.Cout % 8 == 0) launch_bwd_data<true, true, PB, 2>(nt, blocks, st, g, dy, y, slope, pb, wt, dx, accumulate);
            else launch_bwd_data<false, true, PB, 2>(nt, blocks, st, g, dy, y, slope, pb, wt, dx, accumulate);
        } else {
            if (g.Cout % 8 == 0) launch_bwd_data<true, true, PB, 1>(nt, blocks, st, g, dy, y, slope, pb, wt, dx, accumulate);
            else launch_bwd_data<false, true, PB, 1>(nt, blocks, st, g, dy, y, slope, pb, wt, dx, accumulate);
        }
    } else {
        const long long M = (long long)g.N * g.Di * g.Hi * g.Wi;
        const unsigned blocks = (unsigned)((M + 64 * MTv - 1) / (64 * MTv));
        if (MTv == 2) {
            if (g.Cout % 8 == 0) launch_bwd_data<true, false, PB, 2>(nt, blocks, st, g, dy, y, slope, pb, wt, dx, accumulate);
            else launch_bwd_data<false, false, PB, 2>(nt, blocks, st, g, dy, y, slope, pb, wt, dx, accumulate);
        } else {
            if (g.Cout % 8 == 0) launch_bwd_data<true, false, PB, 1>(nt, blocks, st, g, dy, y, slope, pb, wt, dx, accumulate);
            else launch_bwd_data<false, false, PB, 1>(nt, blocks, st, g, dy, y, slope, pb, wt, dx, accumulate);
        }
    }
    return hipGetLastError();
}

hipError_t conv_bwd_data_launch(const ConvGeom& g, const float* dy, const unsigned short* y, float slope,
                                const unsigned short* wt, float* dx, int accumulate, hipStream_t st)
{
    return bwd_data_dispatch<false>(g, dy, y, slope, nullptr, wt, dx, accumulate, st);
}

hipError_t conv_bwd_data_p_launch(const ConvGeom& g, const unsigned short* p, const unsigned short* wt, float* dx,
                                  int accumulate, hipStream_t st)
{
    return bwd_data_dispatch<true>(g, nullptr, nullptr, 0.0f, p, wt, dx, accumulate, st);
}

// P = bf16(dL/dy act'(y)) elementwise (y NULL: the identity), the rounding of
// the operand packing in the backward kernels (round to nearest even).
__global__ void __launch_bounds__(256) act_grad_kernel(const float* __restrict__ dy, const unsigned short* __restrict__ y,
                                                       float slope, long long n, unsigned short* __restrict__ p)
{
    for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < n; i += (long long)gridDim.x * 256) {
        float v = dy[i];
        if (y) v *= lrelu_d(y[i], slope);
        p[i] = f2bf(v);
    }
}

// The same, 8 elements per thread and step (n8 groups of 8; 16-byte aligned
// operands): two 16-byte loads of dy, one of y, one 16-byte store.
__global__ void __launch_bounds__(256) act_grad8_kernel(const float* __restrict__ dy,
                                                        const unsigned short* __restrict__ y, float slope, long long n8,
                                                        unsigned short* __restrict__ p)
{
    for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < n8; i += (long long)gridDim.x * 256) {
        const float4 d0 = reinterpret_cast<const float4*>(dy)[2 * i];
        const float4 d1 = reinterpret_cast<const float4*>(dy)[2 * i + 1];
        float v[8] = {d0.x, d0.y, d0.z, d0.w, d1.x, d1.y, d1.z, d1.w};
        if (y) {
            const uint4 yv = reinterpret_cast<const uint4*>(y)[i];
            const unsigned yw[4] = {yv.x, yv.y, yv.z, yv.w};
#pragma unroll
            for (int q = 0; q < 8; ++q) v[q] *= lrelu_d((unsigned short)(yw[q >> 1] >> (16 * (q & 1))), slope);
        }
        uint4 o;
        o.x = (unsigned)f2bf(v[0]) | ((unsigned)f2bf(v[1]) << 16);
        o.y = (unsigned)f2bf(v[2]) | ((unsigned)f2bf(v[3]) << 16);
        o.z = (unsigned)f2bf(v[4]) | ((unsigned)f2bf(v[5]) << 16);
        o.w = (unsigned)f2bf(v[6]) | ((unsigned)f2bf(v[7]) << 16);
        reinterpret_cast<uint4*>(p)[i] = o;
    }
}

hipError_t act_grad_launch(const float* dy, const unsigned short* y, float slope, long long n, unsigned short* p,
                           hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    const bool a16 = ((reinterpret_cast<uintptr_t>(dy) | reinterpret_cast<uintptr_t>(y) |
                       reinterpret_cast<uintptr_t>(p)) & 15u) == 0;
    long long head = 0;  // elements done by the vector kernel
    if (a16 && n >= 8) {
        const long long n8 = n / 8;
        long long blocks = (n8 + 255) / 256;
        if (blocks > 65536) blocks = 65536;
        hipLaunchKernelGGL(act_grad8_kernel, dim3((unsigned)blocks), dim3(256), 0, st, dy, y, slope, n8, p);
        head = n8 * 8;
    }
    if (head < n) {
        const long long rest = n - head;
        long long blocks = (rest + 255) / 256;
        if (blocks > 65536) blocks = 65536;
        hipLaunchKernelGGL(act_grad_kernel, dim3((unsigned)blocks), dim3(256), 0, st, dy + head, y ? y + head : nullptr,
                           slope, rest, p + head);
    }
    return hipGetLastError();
}

hipError_t cast_bf16_launch(const float* x, long long n, unsigned short* y, hipStream_t st)
{
    hipLaunchKernelGGL(cast_bf16_kernel, dim3(grid_for(n)), dim3(256), 0, st, x, n, y);
    return hipGetLastError();
}

hipError_t weight_prep_launch(const float* w, int Cout, int Cin, unsigned short* wbf, unsigned short* wt,
                              hipStream_t st)
{
    hipLaunchKernelGGL(weight_prep_kernel, dim3(grid_for((long long)Cout * 27 * Cin)), dim3(256), 0, st, w, Cout, Cin,
                       wbf, wt);
    return hipGetLastError();
}

hipError_t pack_pair_launch(const float* F, const float* M, long long nvox, unsigned short* x, hipStream_t st)
{
    hipLaunchKernelGGL(pack_pair_kernel, dim3(grid_for(nvox)), dim3(256), 0, st, F, M, nvox, x);
    return hipGetLastError();
}

hipError_t split_grad_launch(const ConvGeom& g, const float* dxc, float* dxa, float* dxb, int acc_a, int acc_b,
                             hipStream_t st)
{
    const int Rc = g.N * (g.Di >> 1) * (g.Hi >> 1);  // coarse rows: the voxel count is below 2^31
    hipLaunchKernelGGL(split_grad_kernel, dim3((unsigned)Rc), dim3(256), 0, st, g, dxc, dxa, dxb, acc_a, acc_b);
    return hipGetLastError();
}

hipError_t mse_launch(const float* pred, int Cp, const float* tgt, long long nvox_per, int N, float* dpred,
                      double* part, int nblocks, float* loss, hipStream_t st)
{
    const double scale = 1.0 / ((double)nvox_per * N * 3.0);
    hipLaunchKernelGGL(mse_kernel, dim3(nblocks), dim3(256), 0, st, pred, Cp, tgt, nvox_per, N, dpred, part, scale);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (loss) {
        hipLaunchKernelGGL(sum_partials_kernel, dim3(1), dim3(256), 0, st, part, nblocks, loss);
        e = hipGetLastError();
    }
    return e;
}

hipError_t unpack_disp_launch(const float* pred, int Cp, long long nvox_per, int N, float* u, hipStream_t st)
{
    hipLaunchKernelGGL(unpack_disp_kernel, dim3(grid_for(nvox_per * N)), dim3(256), 0, st, pred, Cp, nvox_per, N, u);
    return hipGetLastError();
}

}  // namespace ffdp
