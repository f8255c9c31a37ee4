// Streaming kernels: standalone warp, pyramid resample, Adam.
#include "adam.hpp"
#include "device.hpp"
#include "internal.hpp"

namespace ffdp {

// out(x) = M(x + u(x)) (Alg. gridsampler Forward), one thread per voxel;
// a block covers 256 consecutive x of one row so loads coalesce.
template <int PAD>
__global__ void __launch_bounds__(256) warp_kernel(const float* __restrict__ M, const float* __restrict__ u, int D,
                                                   int H, int W, float* __restrict__ out)
{
    const int x = blockIdx.x * 256 + threadIdx.x;
    const int y = blockIdx.y;
    const int HW = H * W;
    const size_t N = (size_t)D * HW;
    if (x >= W) return;
    for (int z = blockIdx.z; z < D; z += gridDim.z) {
        const int idx = z * HW + y * W + x;
        float ux = 0.f, uy = 0.f, uz = 0.f;
        if (u) { ux = u[idx]; uy = u[N + idx]; uz = u[2 * N + idx]; }
        out[idx] = trilinear<PAD, false>(M, D, H, W, x, y, z, ux, uy, uz).v;
    }
}

hipError_t warp_launch(const float* M, const float* u, int D, int H, int W, int pad, float* out, hipStream_t st)
{
    dim3 grid((W + 255) / 256, H, D < 64 ? D : 64), block(256);
    if (pad == PAD_BORDER) hipLaunchKernelGGL((warp_kernel<PAD_BORDER>), grid, block, 0, st, M, u, D, H, W, out);
    else hipLaunchKernelGGL((warp_kernel<PAD_ZEROS>), grid, block, 0, st, M, u, D, H, W, out);
    return hipGetLastError();
}

// Composite implicit sampler, forward: out(X) = M(X + Am X + t + S u(X)).
template <int PAD>
__global__ void __launch_bounds__(256) warp_affine_kernel(const float* __restrict__ M, const float* __restrict__ u,
                                                          int D, int H, int W, Affine f, float* __restrict__ out)
{
    const int x = blockIdx.x * 256 + threadIdx.x;
    const int y = blockIdx.y;
    const int HW = H * W;
    const size_t N = (size_t)D * HW;
    if (x >= W) return;
    for (int z = blockIdx.z; z < D; z += gridDim.z) {
        const int idx = z * HW + y * W + x;
        float ux = 0.f, uy = 0.f, uz = 0.f;
        if (u) { ux = u[idx]; uy = u[N + idx]; uz = u[2 * N + idx]; }
        float dx, dy, dz;
        affine_disp(f, x, y, z, ux, uy, uz, dx, dy, dz);
        out[idx] = trilinear<PAD, false>(M, D, H, W, x, y, z, dx, dy, dz).v;
    }
}

hipError_t warp_affine_launch(const float* M, const float* u, int D, int H, int W, const Affine& f, int pad,
                              float* out, hipStream_t st)
{
    dim3 grid((W + 255) / 256, H, D < 64 ? D : 64), block(256);
    if (pad == PAD_BORDER) hipLaunchKernelGGL((warp_affine_kernel<PAD_BORDER>), grid, block, 0, st, M, u, D, H, W, f, out);
    else hipLaunchKernelGGL((warp_affine_kernel<PAD_ZEROS>), grid, block, 0, st, M, u, D, H, W, f, out);
    return hipGetLastError();
}

// Composite sampler adjoint for an upstream gradient gout: dL/du = S^T g
// (written when gu is given), and per-block partial sums of g X^T and g,
// g = gout dM/dp, in the MI tiling (64 x 4 columns, z-chunks).
template <int PAD>
__global__ void __launch_bounds__(MI_NT) warp_affine_bwd_kernel(const float* __restrict__ M,
                                                                const float* __restrict__ u, int D, int H, int W,
                                                                Affine f, const float* __restrict__ gout,
                                                                float* __restrict__ gu, double* __restrict__ part,
                                                                int ntx, int nty, int zchunk, int nblocks)
{
    const int bid = xcd_remap(blockIdx.x, nblocks);
    const int tx = bid % ntx, rest = bid / ntx, ty = rest % nty, ch = rest / nty;
    const int x = tx * MI_TX + (threadIdx.x % MI_TX);
    const int y = ty * MI_TY + (threadIdx.x / MI_TX);
    const int zb = ch * zchunk, ze = min(D, zb + zchunk);
    const int HW = H * W;
    const size_t N = (size_t)D * HW;
    const bool active = x < W && y < H;
    double acc[12];
#pragma unroll
    for (int q = 0; q < 12; ++q) acc[q] = 0.0;
    for (int z = zb; active && z < ze; ++z) {
        const int idx = z * HW + y * W + x;
        float ux = 0.f, uy = 0.f, uz = 0.f;
        if (u) { ux = u[idx]; uy = u[N + idx]; uz = u[2 * N + idx]; }
        float dx, dy, dz;
        affine_disp(f, x, y, z, ux, uy, uz, dx, dy, dz);
        const Tri t = trilinear<PAD, true>(M, D, H, W, x, y, z, dx, dy, dz);
        const float go = gout[idx];
        float gx, gy, gz;
        affine_adjoint(f, x, y, z, go * t.dx, go * t.dy, go * t.dz, acc, gx, gy, gz);
        if (gu) {
            gu[idx] = gx;
            gu[N + idx] = gy;
            gu[2 * N + idx] = gz;
        }
    }
    __shared__ double red[MI_NT];
#pragma unroll
    for (int q = 0; q < 12; ++q) {
        const double v = block_sum<MI_NT>(acc[q], red);
        if (threadIdx.x == 0) part[12 * (size_t)blockIdx.x + q] = v;
    }
}

// out[q] = sum_b part[12 b + q] in a fixed order (a block of 256 threads per q;
// one block for all twelve took 16 us for 960 partials)
__global__ void __launch_bounds__(256) affine_reduce_kernel(const double* __restrict__ part, int nblocks,
                                                            double* __restrict__ out)
{
    __shared__ double red[256];
    const int q = blockIdx.x;
    double s = 0.0;
    for (int b = threadIdx.x; b < nblocks; b += 256) s += part[12 * (size_t)b + q];
    s = block_sum<256>(s, red);
    if (threadIdx.x == 0) out[q] = s;
}

hipError_t affine_reduce_launch(const double* part, int nblocks, double* out, hipStream_t st)
{
    hipLaunchKernelGGL(affine_reduce_kernel, dim3(12), dim3(256), 0, st, part, nblocks, out);
    return hipGetLastError();
}

hipError_t warp_affine_bwd_launch(const float* M, const float* u, int D, int H, int W, const Affine& f, int pad,
                                  const float* gout, float* gu, double* part, double* gAt, hipStream_t st)
{
    const MiLaunch L = mi_plan(D, H, W);
    dim3 grid(L.nblocks), block(MI_NT);
    if (pad == PAD_BORDER)
        hipLaunchKernelGGL((warp_affine_bwd_kernel<PAD_BORDER>), grid, block, 0, st, M, u, D, H, W, f, gout, gu, part,
                           L.ntx, L.nty, L.zchunk, L.nblocks);
    else
        hipLaunchKernelGGL((warp_affine_bwd_kernel<PAD_ZEROS>), grid, block, 0, st, M, u, D, H, W, f, gout, gu, part,
                           L.ntx, L.nty, L.zchunk, L.nblocks);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return affine_reduce_launch(part, L.nblocks, gAt, st);
}

// Corner-aligned trilinear resize: dst j samples src at j (n_s - 1)/(n_d - 1).
__global__ void __launch_bounds__(256) resample_kernel(const float* __restrict__ src, int sD, int sH, int sW,
                                                       float* __restrict__ dst, int dD, int dH, int dW, float fz,
                                                       float fy, float fx, float scale)
{
    const int x = blockIdx.x * 256 + threadIdx.x;
    const int y = blockIdx.y;
    const int c = blockIdx.z;
    if (x >= dW) return;
    const float* s = src + (size_t)c * sD * sH * sW;
    float* d = dst + (size_t)c * dD * dH * dW;
    const float px = x * fx, py = y * fy;
    const int x0 = min((int)px, sW - 1), y0 = min((int)py, sH - 1);
    const int x1 = min(x0 + 1, sW - 1), y1 = min(y0 + 1, sH - 1);
    const float ax = px - x0, ay = py - y0;
    for (int z = 0; z < dD; ++z) {
        const float pz = z * fz;
        const int z0 = min((int)pz, sD - 1), z1 = min(z0 + 1, sD - 1);
        const float az = pz - z0;
        const float* r00 = s + ((size_t)z0 * sH + y0) * sW;
        const float* r01 = s + ((size_t)z0 * sH + y1) * sW;
        const float* r10 = s + ((size_t)z1 * sH + y0) * sW;
        const float* r11 = s + ((size_t)z1 * sH + y1) * sW;
        const float c00 = fmaf(ax, r00[x1] - r00[x0], r00[x0]);
        const float c01 = fmaf(ax, r01[x1] - r01[x0], r01[x0]);
        const float c10 = fmaf(ax, r10[x1] - r10[x0], r10[x0]);
        const float c11 = fmaf(ax, r11[x1] - r11[x0], r11[x0]);
        const float c0 = fmaf(ay, c01 - c00, c00), c1 = fmaf(ay, c11 - c10, c10);
        d[((size_t)z * dH + y) * dW + x] = scale * fmaf(az, c1 - c0, c0);
    }
}

hipError_t resample_launch(const float* src, int sD, int sH, int sW, float* dst, int dD, int dH, int dW, int ch,
                           float scale, hipStream_t st)
{
    const float fz = dD > 1 ? (float)((double)(sD - 1) / (double)(dD - 1)) : 0.0f;
    const float fy = dH > 1 ? (float)((double)(sH - 1) / (double)(dH - 1)) : 0.0f;
    const float fx = dW > 1 ? (float)((double)(sW - 1) / (double)(dW - 1)) : 0.0f;
    dim3 grid((dW + 255) / 256, dH, ch), block(256);
    hipLaunchKernelGGL(resample_kernel, grid, block, 0, st, src, sD, sH, sW, dst, dD, dH, dW, fz, fy, fx, scale);
    return hipGetLastError();
}

// Adam, 4 elements per thread when every pointer is 16-byte aligned (the
// float4 path moves 1 KiB per wave instruction), one float4 per thread over
// the whole grid, with non-temporal loads and stores: every byte is touched
// once, so the fields stream past the caches (22% faster than a grid-stride
// loop of 8192 cached blocks on a 3 x 512^3 field).
typedef float f32x4 __attribute__((ext_vector_type(4)));

__global__ void __launch_bounds__(256) adam_vec_kernel(f32x4* __restrict__ x, const f32x4* __restrict__ g,
                                                       f32x4* __restrict__ m, f32x4* __restrict__ v, size_t n4,
                                                       AdamK k)
{
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n4; i += (size_t)gridDim.x * 256) {
        f32x4 xx = __builtin_nontemporal_load(x + i), gg = __builtin_nontemporal_load(g + i);
        f32x4 mm = __builtin_nontemporal_load(m + i), vv = __builtin_nontemporal_load(v + i);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            float a = xx[e], b = mm[e], c = vv[e];
            adam1(a, gg[e], b, c, k);
            xx[e] = a; mm[e] = b; vv[e] = c;
        }
        __builtin_nontemporal_store(xx, x + i);
        __builtin_nontemporal_store(mm, m + i);
        __builtin_nontemporal_store(vv, v + i);
    }
}

__global__ void __launch_bounds__(256) adam_scalar_kernel(float* __restrict__ x, const float* __restrict__ g,
                                                          float* __restrict__ m, float* __restrict__ v, size_t n,
                                                          AdamK k)
{
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) {
        float xx = x[i], mm = m[i], vv = v[i];
        adam1(xx, g[i], mm, vv, k);
        x[i] = xx; m[i] = mm; v[i] = vv;
    }
}

hipError_t adam_launch(float* x, const float* g, float* m, float* v, int64_t n, float lr, float b1, float b2,
                       float eps, int64_t step, hipStream_t st)
{
    const AdamK k = adam_constants(lr, b1, b2, eps, step);
    const bool aligned = ((((uintptr_t)x) | ((uintptr_t)g) | ((uintptr_t)m) | ((uintptr_t)v)) & 15) == 0;
    const size_t nn = (size_t)n;
    size_t done = 0;
    if (aligned && nn >= 4) {
        const size_t n4 = nn / 4;
        size_t blocks = (n4 + 255) / 256;
        if (blocks > 0x7fffffff) blocks = 0x7fffffff;
        hipLaunchKernelGGL(adam_vec_kernel, dim3((unsigned)blocks), dim3(256), 0, st, (f32x4*)x, (const f32x4*)g,
                           (f32x4*)m, (f32x4*)v, n4, k);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        done = n4 * 4;
    }
    if (done < nn) {
        const size_t rem = nn - done;
        size_t blocks = (rem + 255) / 256;
        if (blocks > 8192) blocks = 8192;
        hipLaunchKernelGGL(adam_scalar_kernel, dim3((unsigned)blocks), dim3(256), 0, st, x + done, g + done, m + done,
                           v + done, rem, k);
        return hipGetLastError();
    }
    return hipSuccess;
}

// Checked mode: one flag word set when any value of an input is NaN or
// infinite (exponent bits all ones).  Cleared by a kernel rather than a
// memset, so a captured call records no memset node.
__global__ void __launch_bounds__(64) finite_flag_clear(unsigned* flag)
{
    if (threadIdx.x == 0) *flag = 0u;
}

__global__ void __launch_bounds__(256) finite_check_kernel(const float* __restrict__ p, long long n,
                                                           unsigned* __restrict__ flag)
{
    bool bad = false;
    for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < n; i += (long long)gridDim.x * 256)
        bad |= (__float_as_uint(p[i]) & 0x7f800000u) == 0x7f800000u;
    if (__builtin_amdgcn_ballot_w64(bad) != 0 && (threadIdx.x & 63) == 0) atomicOr(flag, 1u);
}

hipError_t finite_clear_launch(unsigned* flag, hipStream_t st)
{
    hipLaunchKernelGGL(finite_flag_clear, dim3(1), dim3(64), 0, st, flag);
    return hipGetLastError();
}

hipError_t finite_check_launch(const float* p, long long n, unsigned* flag, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    long long blocks = (n + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(finite_check_kernel, dim3((unsigned)blocks), dim3(256), 0, st, p, n, flag);
    return hipGetLastError();
}

}  // namespace ffdp
