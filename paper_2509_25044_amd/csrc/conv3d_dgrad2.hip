// Input gradient of the stride-2 3x3x3 BF16 convolutions (gfx950):
//   dX[i][ci] = sum_{t,co} P[(i + 1 - t) / 2][co] W[co][t][ci]   (integer indices only)
// with P = dL/dy act'(y) in bf16.  FP32 accumulation on v_mfma_f32_16x16x32_bf16.
//
// Along an axis an even input voxel i = 2 I meets tap 1 of output I, an odd
// one i = 2 I + 1 meets tap 2 of output I and tap 0 of output I + 1.  So the 8
// parity classes of the input voxels are sums over P at the 8 shifts (0 or 1
// per axis) of the coarse grid, 27 (class, shift) pairs in all and no
// structural zeros.
//
// A block takes 16 coarse voxels in x, WR * RW rows in y and WN tiles of 16
// input channels, and streams along z.  LDS holds P of three coarse slices
// (two in use, the next one arriving), in 16-byte units of 8 channels,
// [group][chunk][row][x].  A wave owns RW rows of one channel tile and all 8
// classes of them; each P fragment it reads meets every class it belongs to (8
// of them at shift 0).  Weights are the A operand, so a lane holds 4
// consecutive channels of a voxel.
//
// Bound: the write of the fp32 gradient in the first layer (16 <- 32 channels,
// batch of 4 clinical pairs: 0.42 ms, 4.7 TB/s; 2.19 ms with a kernel that
// gathered both operands per lane and parity class), the weight fragments'
// reads in the deeper ones, where each meets RW MFMAs (0.46 -> 0.19 and 0.19 ->
// 0.07 ms).
#include "conv_p.hpp"
#include "conv_tile.hpp"
#include "device.hpp"

namespace ffdp {

namespace {

template <int RW, int WR, int WN, int NG>
struct D2Tile {
    static constexpr int NT = 64 * WR * WN, YT = WR * RW;
    static constexpr int XW = 17, XH = YT + 1;
    static constexpr int PL = XW * XH + ((10 - XW * XH % 8) % 8);  // plane of a chunk, 2 (mod 8) units
    static constexpr int GU = XW * XH * 4;                         // staged units of a group
    static constexpr int NU = (GU * NG + NT - 1) / NT;
    static constexpr bool WLDS = NG == 1 && WN == 1;               // weights resident
    static constexpr int WB = WLDS ? 27 * 64 * WN : 0;
};

// tap along one axis of parity p at shift s; -1: none
__host__ __device__ constexpr int d2_tap(int p, int s) { return p == 0 ? (s == 0 ? 1 : -1) : (s == 0 ? 2 : 0); }

// NG: the most groups of 32 output channels
template <int RW, int WR, int WN, int NG, bool FROMDY>
__global__ void __launch_bounds__(64 * WR * WN, 2) conv_dgrad2_kernel(TcArgs a)
{
    using T = D2Tile<RW, WR, WN, NG>;
    extern __shared__ uint4 lds[];
    uint4* const ps = lds + T::WB;  // [3][ng][4][PL]
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wn = wave % WN, wr = wave / WN;
    int q = xcd_remap(blockIdx.x, a.nblocks);
    const int n0 = (q % a.nnb) * WN * 16; q /= a.nnb;
    const int x0 = (q % a.nx) * 16; q /= a.nx;
    const int y0 = (q % a.ny) * T::YT; q /= a.ny;
    const int z0 = (q % a.nz) * a.zlen;
    const int bn = q / a.nz;
    const int z1 = min(a.Do, z0 + a.zlen);
    const int C = a.Ca;
    const bool c8 = (C & 7) == 0;
    const bool active = n0 + wn * 16 < a.Nout && y0 + wr * RW < a.Ho;
    const int sb = a.ng * 4 * T::PL;  // units of a slice buffer

    // 8 weights of lane l: input channel n, channels 8 (l / 16) .. of group g, tap
    auto weight = [&](int g, int tap, int l, int tile) __attribute__((always_inline)) {
        const int n = n0 + tile * 16 + (l & 15), c = 32 * g + 8 * (l >> 4);
        const gptr p = as_global(a.w) + ((size_t)n * 27 + tap) * C + c, z = as_global(&tc_zero);
        const bool ok = n < a.Nout && c < C;
        if (c8) return ld16(ok ? p : z);
        const uint2 lo = ld8(ok ? p : z), hi = ld8(ok && c + 8 <= C ? p + 4 : z);
        return make_uint4(lo.x, lo.y, hi.x, hi.y);
    };
    if constexpr (T::WLDS)
        for (int p = tid; p < T::WB; p += T::NT) lds[p] = weight(0, p >> 6, p & 63, 0);

    uint4 xr[T::NU];
    auto load = [&](int zc) __attribute__((always_inline)) {
        const bool zok = zc < a.Do;
        const size_t base = ((size_t)bn * a.Do + (zok ? zc : 0)) * ((size_t)a.Ho * a.Wo) * C;
        const int t0 = opaque(tid);
        const gptr z = as_global(&tc_zero), src = as_global(a.xa);
#pragma unroll
        for (int u = 0; u < T::NU; ++u) {
            const int p = t0 + T::NT * u, v = p >> 2;  // chunks of a voxel, voxels, groups
            const int g = v / (T::XW * T::XH), vg = v - g * (T::XW * T::XH);
            const int vy = vg / T::XW, X = x0 + vg - vy * T::XW, Y = y0 + vy, c = 32 * g + 8 * (p & 3);
            const bool ok = zok && g < a.ng && c < C && X < a.Wo && Y < a.Ho;
            const size_t o = base + (size_t)(unsigned)(Y * a.Wo + X) * C;
            uint4 r = make_uint4(0u, 0u, 0u, 0u);
            if constexpr (FROMDY) {
                if (ok) r = p_from_dy8(a.dy, a.y, a.slope, o, c, C);
            } else if (c8) {
                r = ld16(ok ? src + o + c : z);
            } else {
                const uint2 lo = ld8(ok ? src + o + c : z), hi = ld8(ok && c + 8 <= C ? src + o + c + 4 : z);
                r = make_uint4(lo.x, lo.y, hi.x, hi.y);
            }
            xr[u] = r;
        }
    };
    auto store = [&](int buf) __attribute__((always_inline)) {
        const int t0 = opaque(tid);
#pragma unroll
        for (int u = 0; u < T::NU; ++u) {
            const int p = t0 + T::NT * u, v = p >> 2;
            const int g = v / (T::XW * T::XH), vg = v - g * (T::XW * T::XH);
            if (g < a.ng) ps[buf * sb + (4 * g + (p & 3)) * T::PL + vg] = xr[u];
        }
    };

    load(z0);
    store(0);
    load(z0 + 1);
    store(1);
    __syncthreads();
    int b0 = 0;  // buffer of slice zc
    for (int zc = z0; zc < z1; ++zc) {
        const int b1 = b0 == 2 ? 0 : b0 + 1, b2 = b1 == 2 ? 0 : b1 + 1;
        const bool more = zc + 1 < z1;
        if (more) load(zc + 2);
        if (active) {
            f4v acc[2][2][2][RW];
#pragma unroll
            for (int e = 0; e < 8 * RW; ++e) acc[e & 1][(e >> 1) & 1][(e >> 2) & 1][e >> 3] = f4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
            for (int g = 0; g < a.ng; ++g) {
                const int lane = opaque(tid & 63);
                // the 27 weights in blocks of one (sz, sx, pz), 3 or 6 each: (py, sy) fastest
                constexpr int BZ[6] = {0, 0, 0, 0, 1, 1}, BX[6] = {0, 0, 1, 1, 0, 1}, BP[6] = {0, 1, 0, 1, 1, 1};
                uint4 w[2][6];
                auto weights = [&](int b, uint4* o) __attribute__((always_inline)) {
#pragma unroll
                    for (int e = 0; e < 6; ++e) {
                        const int px = BX[b] ? 1 : e / 3, py = e % 3 > 0, sy = e % 3 > 1;
                        if (BX[b] && e >= 3) break;
                        const int tap = d2_tap(BP[b], BZ[b]) * 9 + d2_tap(py, sy) * 3 + d2_tap(px, BX[b]);
                        o[e] = T::WLDS ? lds[tap * 64 + lane] : weight(g, tap, lane, wn);
                    }
                };
                weights(0, w[0]);
                uint4 P[RW + 1];
#pragma unroll
                for (int b = 0; b < 6; ++b) {
                    __builtin_amdgcn_sched_barrier(0);
                    if (b + 1 < 6) weights(b + 1, w[(b + 1) & 1]);
                    if (b == 0 || BX[b] != BX[b - 1] || BZ[b] != BZ[b - 1]) {
                        const uint4* const p = ps + (BZ[b] ? b1 : b0) * sb + (4 * g + (lane >> 4)) * T::PL +
                                               wr * RW * T::XW + (lane & 15) + BX[b];
#pragma unroll
                        for (int r = 0; r <= RW; ++r) P[r] = p[r * T::XW];
                    }
#pragma unroll
                    for (int e = 0; e < 6; ++e) {
                        const int px = BX[b] ? 1 : e / 3, py = e % 3 > 0, sy = e % 3 > 1;
                        if (BX[b] && e >= 3) break;
#pragma unroll
                        for (int r = 0; r < RW; ++r)
                            acc[BP[b]][py][px][r] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                                as_bf8(w[b & 1][e]), as_bf8(P[r + sy]), acc[BP[b]][py][px][r], 0, 0, 0);
                    }
                }
            }
            const int lane = opaque(tid & 63), ci = n0 + wn * 16 + 4 * (lane >> 4), x = 2 * (x0 + (lane & 15));
            if (ci < a.Nout) {
#pragma unroll
                for (int pz = 0; pz < 2; ++pz)
#pragma unroll
                    for (int r = 0; r < RW; ++r)
#pragma unroll
                        for (int py = 0; py < 2; ++py) {
                            const int z = 2 * zc + pz, y = 2 * (y0 + wr * RW + r) + py;
                            if (z >= a.Di || y >= a.Hi) continue;
                            float* const d = a.yf + ((((size_t)bn * a.Di + z) * a.Hi + y) * a.Wi + x) * a.Nout + ci;
#pragma unroll
                            for (int px = 0; px < 2; ++px) {
                                if (x + px >= a.Wi) continue;
                                f32x4_a4* const dp = reinterpret_cast<f32x4_a4*>(d + px * a.Nout);
                                const f4v v = acc[pz][py][px][r];
                                f32x4_a4 o = {v[0], v[1], v[2], v[3]};
                                if (a.accumulate) o += *dp;
                                *dp = o;
                            }
                        }
            }
        }
        if (more) store(b2);
        b0 = b1;
        __syncthreads();
    }
}

template <int RW, int WR, int WN, int NG, bool FROMDY>
hipError_t d2_launch(TcArgs& a, hipStream_t st)
{
    using T = D2Tile<RW, WR, WN, NG>;
    const int lds = (T::WB + 3 * a.ng * 4 * T::PL) * 16;
    const hipError_t e = tc_plan(a, a.Do, a.Ho, a.Wo, T::YT, WN, lds <= TC_LDS / 2 ? 2 : 1);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((conv_dgrad2_kernel<RW, WR, WN, NG, FROMDY>), dim3((unsigned)a.nblocks), dim3(T::NT), lds, st, a);
    return hipGetLastError();
}

// A wave per tile of 16 input channels; the waves left over split rows, as far
// as three slices of all the groups fit LDS beside a second block.
template <bool FROMDY>
hipError_t d2_dispatch(TcArgs& a, hipStream_t st)
{
    const int nt = (a.Nout + 15) / 16;
    if (nt == 1 && a.ng == 1) return d2_launch<2, 4, 1, 1, FROMDY>(a, st);
    if (nt <= 2 && a.ng <= 2) return d2_launch<4, 2, 2, 2, FROMDY>(a, st);
    return d2_launch<4, 1, 4, 4, FROMDY>(a, st);
}

}  // namespace

hipError_t conv_dgrad2_launch(const ConvGeom& g, const float* dy, const unsigned short* y, float slope,
                              const unsigned short* pb, const unsigned short* wt, float* dx, int accumulate,
                              hipStream_t st)
{
    TcArgs a{};
    a.N = g.N; a.Di = g.Di; a.Hi = g.Hi; a.Wi = g.Wi; a.Do = g.Do; a.Ho = g.Ho; a.Wo = g.Wo;
    a.Ca = g.Cout; a.Nout = g.Ca + g.Cb;
    a.xa = pb; a.dy = dy; a.y = y; a.slope = slope; a.w = wt; a.yf = dx; a.accumulate = accumulate;
    a.na = a.ng = (g.Cout + 31) / 32;
    return pb ? d2_dispatch<false>(a, st) : d2_dispatch<true>(a, st);
}

}  // namespace ffdp
