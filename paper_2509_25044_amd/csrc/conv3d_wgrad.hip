// Weight and bias gradient of the 3x3x3 BF16 convolutions (stride 1 or 2), gfx950:
//   dW[co][t][ci] = sum_o P[o][co] X[o s + t - 1][ci],   db[co] = sum_o P[o][co]
// with P = dL/dy act'(y) rounded to bf16.
//
// The product's K dimension is output voxels, but the tensors are
// channels-last, so both operands need a transpose: ds_read_b64_tr_b16 reads
// 4 voxels x 16 channels from LDS with the lanes of a 16-lane group holding
// one channel each, which is the operand layout of
// v_mfma_f32_16x16x32_bf16 (two such reads give a lane 8 consecutive voxels
// of its channel).  LDS therefore keeps the natural [voxel][16 channels]
// order, written with 16-byte stores, and a tap's shift is an address.
//
// A block takes one tile of 16 output channels, one tile of 16 input channels
// and a chunk of columns: 32 x (4 RW) output voxels in x, y, streamed along z.
// Per input slice it stages the slice with its halo (the next one's loads are
// in flight meanwhile) and one slice of P.  Wave w owns RW output rows and all
// 27 taps: the P fragments of the last three output slices stay in registers,
// and each X fragment (one input row at one of the three x shifts) feeds every
// (dz, dy) tap that pairs it with one of them (stride 1: 12 X and 2 P
// fragment reads for 54 MFMAs).  The bias gradient is one more MFMA per P
// fragment, against ones, in the blocks of the first input-channel tile.  The
// four waves' sums are added in wave order at the end of the chunk.
//
// Channel counts that are not multiples of 16 are padded with zeros in LDS.
//
// Bound: matrix issue at the full-resolution decoder layer (MFMA busy 0.39 of
// the SIMD cycles, two blocks of 4 waves per CU at 239 VGPRs), staging at the
// others.  Clinical batch of 4, 48 -> 16 channels: 1.19 ms (960 TFLOP/s)
// against 5.26 ms of a kernel that wrote X and three shifted copies of P
// transposed into LDS 2 bytes at a time and read both operands for every
// MFMA; 16 -> 32 stride 2: 0.46 against 2.41 ms plus a 0.19 ms transpose of
// P; the bias gradient had been a pass of its own over P (0.15 and 0.04 ms).
#include "conv_types.hpp"
#include "conv_wgrad.hpp"
#include "device.hpp"
#include "internal.hpp"

namespace ffdp {

namespace {

constexpr int WG_X = 32;  // output voxels of a K step

template <int S, int RW>
struct WgTile {
    static constexpr int YT = 4 * RW;                 // output rows per block
    static constexpr int XW = S * (WG_X - 1) + 3;     // input row with halo
    static constexpr int XH = S * (YT - 1) + 3;
    static constexpr int UXW = S * WG_X / 2 + 2, UXH = S * YT / 2 + 2;  // coarse tile of an upsampled part
    static constexpr int NX = (XW * XH * 2 + 255) / 256;        // 16-byte units per thread and slice
    static constexpr int NP = (YT * WG_X * 2 + 255) / 256;
    static constexpr int XS = XW * XH * 16, PS = YT * WG_X * 16;  // shorts per buffer
    static constexpr int LDS = 2 * (XS + PS) * 2;                 // bytes
    static_assert(LDS >= 28 * 64 * 16, "the final reduction reuses the buffers");
    static_assert(S == 1 || RW == 1, "stride 2 takes one output row per wave");
};

typedef __attribute__((address_space(3))) s4v lds_s4v;

// 8 voxels of the lane's channel: two transposing reads at p and q
__device__ __forceinline__ bf8v tr8(const unsigned short* p, const unsigned short* q)
{
    const s4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4v*)(p));
    const s4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4v*)(q));
    return __builtin_bit_cast(bf8v, (s8v)__builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

struct WgArgs {
    ConvGeom g;
    const unsigned short* xa;
    const unsigned short* xb;
    const unsigned short* pbf;  // P, or NULL: from dy and y
    const float* dy;
    const unsigned short* y;
    float slope;
    float* part;
    ConvWgradPlan p;
    int tna, items, nblocks;  // channel tiles of part a; (input, output) tile pairs
};

// CUT: the output's width is not a multiple of 32 (the reads that clear the
// columns past it cost 1 to 2% at stride 1)
template <int S, int RW, bool FROMDY, bool CUT>
__global__ void __launch_bounds__(256, 2) conv_wgrad_kernel(WgArgs a)
{
    using T = WgTile<S, RW>;
    __shared__ __attribute__((aligned(16))) unsigned char lds[T::LDS + 16];
    unsigned short* const xsl = reinterpret_cast<unsigned short*>(lds);  // [2][XS]
    unsigned short* const psl = xsl + 2 * T::XS;                         // [2][PS]
    unsigned short* const zeros = psl + 2 * T::PS;                       // 8 bytes
    const ConvGeom& g = a.g;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int li = lane & 15, kg = lane >> 4;
    const int Cin = g.Ca + g.Cb;
    if (tid < 4) zeros[tid] = 0;
    // the items of one chunk share its voxels: next to each other, on one XCD
    const int bid = xcd_remap(blockIdx.x, a.nblocks);
    const int item = bid % a.items, chunk = bid / a.items;
    const int tn = a.tna + (g.Cb + 15) / 16;
    const int it = item % tn, co0 = (item / tn) * 16;
    const bool pa = it < a.tna;
    const bool ups = pa && g.ups;
    const unsigned short* const xsrc = pa ? a.xa : a.xb;
    const int C = pa ? g.Ca : g.Cb;
    const int cc = (pa ? it : it - a.tna) * 16;    // first channel within the part
    const int ci0 = pa ? cc : g.Ca + cc;           // ... and within the concatenation
    const int sW = ups ? g.Wi >> 1 : g.Wi, sH = ups ? g.Hi >> 1 : g.Hi, sD = ups ? g.Di >> 1 : g.Di;

    // lane addresses of the X fragments: row r of the wave's input rows, shift dx
    const int xpitch = (ups ? T::UXW : T::XW) * 16;
    int xoff[3], xstep[3];
#pragma unroll
    for (int dx = 0; dx < 3; ++dx) {
        const int v0 = S * (8 * kg + (li >> 2)) + dx, v1 = v0 + 4 * S;
        const int u0 = ups ? (v0 + 1) >> 1 : v0, u1 = ups ? (v1 + 1) >> 1 : v1;
        xoff[dx] = u0 * 16 + (li & 3) * 4;
        xstep[dx] = (u1 - u0) * 16;
    }
    constexpr int XR = S * (RW - 1) + 3;  // input rows of a wave
    const int poff = (wave * RW * WG_X + 8 * kg + (li >> 2)) * 16 + (li & 3) * 4;

    f4v acc[3][3][3], accb = f4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int q = 0; q < 27; ++q) acc[q / 9][(q / 3) % 3][q % 3] = f4v{0.f, 0.f, 0.f, 0.f};
    const s8v ones_s = {0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80};
    const bf8v ones = __builtin_bit_cast(bf8v, ones_s);

    const long long ub = (long long)chunk * a.p.upc, ue = min(a.p.units, ub + a.p.upc);
    for (long long unit = ub; unit < ue; ++unit) {
        long long q = unit;
        const int x0 = (int)(q % a.p.nx) * WG_X; q /= a.p.nx;
        const int y0 = (int)(q % a.p.ny) * T::YT; q /= a.p.ny;
        const int z0 = (int)(q % a.p.nz) * a.p.zlen;
        const int n = (int)(q / a.p.nz);
        const int z1 = min(g.Do, z0 + a.p.zlen);
        const int nk = S * (z1 - z0 - 1) + 3;  // input slices S z0 - 1 ..
        // Rows and columns past the output have P = 0, but the first of each would still meet the input's last row or
        // column (tap 0), and 0 times an infinite value is not 0: such a row is skipped, such columns of X are read
        // from zeros.
        const int nrow = g.Ho - y0 - wave * RW;
        const bool past0 = x0 + 8 * kg + (li >> 2) >= g.Wo, past1 = x0 + 8 * kg + (li >> 2) + 4 >= g.Wo;
        const int pitch0 = past0 ? 0 : xpitch, pitch1 = past1 ? 0 : xpitch;

        // this thread's units of a slice: voxel offset in the slice (-1: outside) and LDS slot
        int xv[T::NX], pv[T::NP];
#pragma unroll
        for (int u = 0; u < T::NX; ++u) {
            const int p = tid + 256 * u, v = p >> 1;
            const int w = ups ? T::UXW : T::XW, h = ups ? T::UXH : T::XH;
            const int vx = v % w, vy = v / w;
            const int X = (S * x0 >> (ups ? 1 : 0)) - 1 + vx, Y = (S * y0 >> (ups ? 1 : 0)) - 1 + vy;
            xv[u] = (vy < h && (unsigned)X < (unsigned)sW && (unsigned)Y < (unsigned)sH) ? Y * sW + X : -1;
        }
#pragma unroll
        for (int u = 0; u < T::NP; ++u) {
            const int v = (tid + 256 * u) >> 1;
            const int X = x0 + v % WG_X, Y = y0 + v / WG_X;
            pv[u] = (v < T::YT * WG_X && X < g.Wo && Y < g.Ho) ? Y * g.Wo + X : -1;
        }
        uint4 xr[T::NX], pr[T::NP];
        P8 raw[FROMDY ? T::NP : 1];  // dy and y of the units, P once they are written to LDS
        const int c8 = 8 * (tid & 1);
        auto load_x = [&](int k) {
            const int zf = S * z0 - 1 + k;
            const int zi = ups ? zf >> 1 : zf;
            const bool zok = (unsigned)zi < (unsigned)sD;
            const size_t base = ((size_t)n * sD + (zok ? zi : 0)) * ((size_t)sH * sW);
#pragma unroll
            for (int u = 0; u < T::NX; ++u) {
                xr[u] = make_uint4(0u, 0u, 0u, 0u);
                if (zok && xv[u] >= 0) xr[u] = load_c8(xsrc + (base + xv[u]) * C, cc + c8, C);
            }
        };
        auto load_p = [&](int zo) {
            const size_t base = ((size_t)n * g.Do + zo) * ((size_t)g.Ho * g.Wo);
#pragma unroll
            for (int u = 0; u < T::NP; ++u) {
                pr[u] = make_uint4(0u, 0u, 0u, 0u);
                if constexpr (FROMDY) raw[u] = P8();
                if (pv[u] < 0) continue;
                const size_t o = (base + pv[u]) * g.Cout;
                const int c = co0 + c8;
                if constexpr (FROMDY) {
                    raw[u] = p8_load(a.dy, a.y, o, c, g.Cout);
                } else {
                    pr[u] = load_c8(a.pbf + o, c, g.Cout);
                }
            }
        };
        // input slice k brings output slice z0 + k / S when k % S == 0 (its tap dz = 0)
        auto has_p = [&](int k) { return k % S == 0 && z0 + k / S < z1; };
        auto store = [&](int k) {
            unsigned short* const xd = xsl + (k & 1) * T::XS;
            unsigned short* const pd = psl + (k & 1) * T::PS;
#pragma unroll
            for (int u = 0; u < T::NX; ++u) {
                const int p = tid + 256 * u;
                if (p < T::XW * T::XH * 2) *reinterpret_cast<uint4*>(xd + p * 8) = xr[u];
            }
            if (has_p(k))
#pragma unroll
                for (int u = 0; u < T::NP; ++u) {
                    const int p = tid + 256 * u;
                    if constexpr (FROMDY) pr[u] = p8_form(raw[u], a.y != nullptr, a.slope);
                    if (p < T::YT * WG_X * 2) *reinterpret_cast<uint4*>(pd + p * 8) = pr[u];
                }
        };

        bf8v P[3][RW];  // P of output slices z0 + k / S - 0, 1, 2
#pragma unroll
        for (int d = 0; d < 3; ++d)
#pragma unroll
            for (int r = 0; r < RW; ++r) P[d][r] = ones;  // set before use
        load_x(0);
        load_p(z0);
        store(0);
        __syncthreads();
        for (int k = 0; k < nk; ++k) {
            if (k + 1 < nk) {
                load_x(k + 1);
                if (has_p(k + 1)) load_p(z0 + (k + 1) / S);
            }
            const unsigned short* const xb = xsl + (k & 1) * T::XS;
            const unsigned short* const c0 = past0 ? zeros : xb + xoff[0];  // columns of shift 0
            const unsigned short* const c1 = past1 ? zeros : xb + xoff[0] + xstep[0];
            if (k % S == 0) {  // a new output slice (or the end: the ring still moves)
#pragma unroll
                for (int r = 0; r < RW; ++r) {
                    P[2][r] = P[1][r];
                    P[1][r] = P[0][r];
                }
                if (has_p(k)) {
                    const unsigned short* const pb = psl + (k & 1) * T::PS + poff;
#pragma unroll
                    for (int r = 0; r < RW; ++r) {
                        P[0][r] = tr8(pb + r * WG_X * 16, pb + r * WG_X * 16 + 64);
                        if (it == 0) accb = __builtin_amdgcn_mfma_f32_16x16x32_bf16(P[0][r], ones, accb, 0, 0, 0);
                    }
                }
            }
            // output slices the taps of this input slice pair with (uniform):
            // stride 1: dz -> z0 + k - dz;  stride 2: even k: dz = 0 and 2, odd k: dz = 1
            bool use[3];
#pragma unroll
            for (int dz = 0; dz < 3; ++dz) {
                const int t = k - dz;
                use[dz] = t >= 0 && t % S == 0 && z0 + t / S < z1;
            }
#pragma unroll
            for (int r = 0; r < XR; ++r) {
                // stride 1: input row RW wave + r (coarse (. + 1) / 2); stride 2: 2 wave + r
                const int row = S * RW * wave + r;
                const int urow = ups ? (row + 1) >> 1 : row;
                const unsigned short* const rp = xb + urow * xpitch;
                bf8v X[3];
#pragma unroll
                for (int dx = 0; dx < 3; ++dx) {
                    const unsigned short* const p = rp + xoff[dx];
                    X[dx] = CUT && dx == 0 ? tr8(c0 + __mul24(urow, pitch0), c1 + __mul24(urow, pitch1))
                                           : tr8(p, p + xstep[dx]);
                }
#pragma unroll
                for (int dz = 0; dz < 3; ++dz) {
                    if (!use[dz]) continue;
                    const int d = S == 1 ? dz : dz / 2;  // stride 2: slices k/2 (dz = 0, 1) and k/2 - 1 (dz = 2)
#pragma unroll
                    for (int yo = 0; yo < RW; ++yo) {
                        const int dyy = r - S * yo;
                        if (dyy < 0 || dyy > 2 || (dyy == 0 && yo >= nrow)) continue;
#pragma unroll
                        for (int dx = 0; dx < 3; ++dx)
                            acc[dz][dyy][dx] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(P[d][yo], X[dx],
                                                                                      acc[dz][dyy][dx], 0, 0, 0);
                    }
                }
            }
            if (k + 1 < nk) store(k + 1);
            __syncthreads();
        }
    }

    // add the waves' sums in wave order; wave 3 ends up with the total
    f4v* const red = reinterpret_cast<f4v*>(lds);  // [28][64]
    for (int w = 0; w < 4; ++w) {
        if (wave == w) {
#pragma unroll
            for (int t = 0; t < 28; ++t) {
                f4v v = t < 27 ? acc[(t / 9) % 3][(t / 3) % 3][t % 3] : accb;
                if (w) v += red[t * 64 + lane];
                red[t * 64 + lane] = v;
            }
        }
        __syncthreads();
    }
    // lane of a fragment: co = co0 + 4 kg + e, ci = li
    float* const out = a.part + (size_t)chunk * g.Cout * 27 * Cin;
    const bool civ = cc + li < C;
    for (int t = wave; t < 27; t += 4) {
        const f4v v = red[t * 64 + lane];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int co = co0 + 4 * kg + e;
            if (civ && co < g.Cout) out[((size_t)co * 27 + t) * Cin + ci0 + li] = v[e];
        }
    }
    if (it == 0 && wave == 0 && li == 0) {
        float* const bp = a.part + (size_t)a.p.nchunks * g.Cout * 27 * Cin + (size_t)chunk * g.Cout;
        const f4v v = red[27 * 64 + lane];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int co = co0 + 4 * kg + e;
            if (co < g.Cout) bp[co] = v[e];
        }
    }
}

// dW[q] = sum_c part[c][q], dW fp32.  A block takes 64 consecutive q; its 4
// waves sum the parts c = w, w + 4, ... (w = wave) with 8 loads in flight,
// then the 4 wave sums are added in wave order (a fixed order throughout).
__global__ void __launch_bounds__(256) reduce_parts_kernel(const float* __restrict__ part, int nparts, long long q_n,
                                                           float* __restrict__ out)
{
    __shared__ float red[4][64];
    const int l = (int)threadIdx.x & 63, w = (int)threadIdx.x >> 6;
    const long long q = (long long)blockIdx.x * 64 + l;
    float s = 0.f;
    if (q < q_n) {
        const float* src = part + q;
        int c = w;
        for (; c + 28 < nparts; c += 32) {
            float v[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) v[k] = src[(size_t)(c + 4 * k) * q_n];
#pragma unroll
            for (int k = 0; k < 8; ++k) s += v[k];
        }
        for (; c < nparts; c += 4) s += src[(size_t)c * q_n];
    }
    red[w][l] = s;
    __syncthreads();
    if (w == 0 && q < q_n) out[q] = ((red[0][l] + red[1][l]) + red[2][l]) + red[3][l];
}

constexpr int WG_RW1 = 2, WG_RW2 = 1;  // output rows per wave, stride 1 and 2

template <int S, int RW, bool FROMDY>
void wgrad_kernel_launch(const WgArgs& a, dim3 grid, dim3 block, hipStream_t st)
{
    if (a.g.Wo % WG_X) hipLaunchKernelGGL((conv_wgrad_kernel<S, RW, FROMDY, true>), grid, block, 0, st, a);
    else hipLaunchKernelGGL((conv_wgrad_kernel<S, RW, FROMDY, false>), grid, block, 0, st, a);
}

int wg_items(const ConvGeom& g)
{
    return ((g.Ca + 15) / 16 + (g.Cb + 15) / 16) * ((g.Cout + 15) / 16);
}

}  // namespace

// About 2048 blocks over (chunk, channel tile pairs).  A unit is one column
// over zlen output slices; columns are cut along z only where there are too
// few of them (a cut re-reads two input slices).
ConvWgradPlan conv_wgrad_plan(const ConvGeom& g)
{
    ConvWgradPlan p;
    p.nx = (g.Wo + WG_X - 1) / WG_X;
    const int yt = 4 * (g.stride == 1 ? WG_RW1 : WG_RW2);
    p.ny = (g.Ho + yt - 1) / yt;
    const long long cols = (long long)g.N * p.nx * p.ny;
    const int items = wg_items(g);
    const long long want = (2048 + items - 1) / items;
    long long nz = (want + cols - 1) / cols;
    // Chunks of at least 8 slices; of 2 where those make fewer than 8 blocks, each a
    // chain of its slices (16 -> 16 channels at 8 x 8 x 8: 23.5 -> 18.3 us, from fp32
    // dy 31 -> 19).
    const int zmin = cols * ((g.Do + 7) / 8) * items < 8 ? 2 : 8;
    if (nz > (g.Do + zmin - 1) / zmin) nz = (g.Do + zmin - 1) / zmin;
    p.zlen = (int)((g.Do + nz - 1) / nz);
    p.nz = (g.Do + p.zlen - 1) / p.zlen;
    p.units = cols * p.nz;
    const long long chunks = want < p.units ? want : p.units;
    p.upc = (p.units + chunks - 1) / chunks;
    p.nchunks = (int)((p.units + p.upc - 1) / p.upc);
    p.part_floats = (long long)p.nchunks * g.Cout * (27LL * (g.Ca + g.Cb) + 1);
    return p;
}

hipError_t conv_wgrad_launch(const ConvGeom& g, const unsigned short* xa, const unsigned short* xb, const float* dy,
                             const unsigned short* y, float slope, const unsigned short* pbf, float* dw, float* db,
                             float* part, hipStream_t st)
{
    WgArgs a{};
    a.g = g; a.xa = xa; a.xb = xb; a.pbf = pbf; a.dy = dy; a.y = y; a.slope = slope; a.part = part;
    a.p = conv_wgrad_plan(g);
    a.tna = (g.Ca + 15) / 16;
    a.items = wg_items(g);
    const long long nb = (long long)a.p.nchunks * a.items;
    if (nb > 0x7fffffffLL) return hipErrorInvalidValue;
    a.nblocks = (int)nb;
    const dim3 grid((unsigned)nb), block(256);
    if (g.stride == 1) {
        if (pbf) wgrad_kernel_launch<1, WG_RW1, false>(a, grid, block, st);
        else wgrad_kernel_launch<1, WG_RW1, true>(a, grid, block, st);
    } else {
        if (pbf) wgrad_kernel_launch<2, WG_RW2, false>(a, grid, block, st);
        else wgrad_kernel_launch<2, WG_RW2, true>(a, grid, block, st);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const long long q = (long long)g.Cout * 27 * (g.Ca + g.Cb);
    hipLaunchKernelGGL(reduce_parts_kernel, dim3((unsigned)((q + 63) / 64)), dim3(256), 0, st, part, a.p.nchunks, q, dw);
    if ((e = hipGetLastError()) != hipSuccess || !db) return e;
    hipLaunchKernelGGL(reduce_parts_kernel, dim3((unsigned)((g.Cout + 63) / 64)), dim3(256), 0, st,
                       part + (size_t)a.p.nchunks * q, a.p.nchunks, (long long)g.Cout, db);
    return hipGetLastError();
}

}  // namespace ffdp
