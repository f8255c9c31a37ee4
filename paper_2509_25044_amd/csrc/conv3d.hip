// Small kernels of the warm-start U-Net's training step and the entry points
// of the convolutions' input gradient (gfx950).  Activations are
// channels-last bf16 [N][D][H][W][C].
#include "device.hpp"
#include "internal.hpp"
#include "conv_p.hpp"
#include "conv_types.hpp"

namespace ffdp {

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

hipError_t conv_bwd_data_launch(const ConvGeom& g, const float* dy, const unsigned short* y, float slope,
                                const unsigned short* wt, float* dx, int accumulate, hipStream_t st)
{
    return (g.stride == 1 ? conv_dgrad1_launch : conv_dgrad2_launch)(g, dy, y, slope, nullptr, wt, dx, accumulate, st);
}

hipError_t conv_bwd_data_p_launch(const ConvGeom& g, const unsigned short* p, const unsigned short* wt, float* dx,
                                  int accumulate, hipStream_t st)
{
    return (g.stride == 1 ? conv_dgrad1_launch : conv_dgrad2_launch)(g, nullptr, nullptr, 0.0f, p, wt, dx, accumulate,
                                                                     st);
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
