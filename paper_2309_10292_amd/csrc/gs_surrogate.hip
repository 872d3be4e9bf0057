// Learned 16-step surrogate: a 4-layer 3x3x3 circular convolution network
// (channels 4 -> 32 -> 32 -> 32 -> 2, GELU, residual output) on gfx950 with
// BF16 weights and activations and FP32 accumulation on the matrix cores.
//
// Activations are channels-last (cell-major, channels contiguous: 8 channels
// for the input layer, 32 for hidden layers), so one lane's K fragment of an
// implicit GEMM (8 consecutive channels of one neighbour cell) is one 16-byte
// load. Convolutions are implicit GEMMs with M = cells (tiles of 16 cells of
// one x-row), N = output channels (tiles of 16) and K = 27 offsets x input
// channels, walked in chunks of 32 with v_mfma_f32_16x16x32_bf16 (the output
// layer has its own form); the packed weights of a layer sit in registers or LDS. The data gradient is the same convolution
// with the weights transposed and the offsets mirrored; the weight gradient
// is a GEMM with K = cells, reduced per workgroup into FP32 partials.
#include "gs_device.hpp"
#include "gs_surrogate.hpp"

#include <algorithm>

namespace gs {
namespace nn {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4))); // a native vector (no struct copies)
typedef uint16_t u16;

__device__ __forceinline__ float bf2f(u16 b) { return __uint_as_float((uint32_t)b << 16); }
__device__ __forceinline__ u16 f2bf(float f) { return bf16_rne(f).bits; }

// erf(x) / 2 by Abramowitz and Stegun 7.1.26 (Hastings' rational approximation, here
// with half its coefficients; |error of erf| <= 1.5e-7, far below the BF16 rounding
// of the activations), without branches; e receives exp(-x^2), which the GELU's
// derivative reuses.
__device__ __forceinline__ float half_erf(float x, float &e)
{
    const float ax = fabsf(x);
    const float t = __builtin_amdgcn_rcpf(__builtin_fmaf(0.3275911f, ax, 1.0f));
    float p = __builtin_fmaf(0.5f * 1.061405429f, t, 0.5f * -1.453152027f);
    p = __builtin_fmaf(p, t, 0.5f * 1.421413741f);
    p = __builtin_fmaf(p, t, 0.5f * -0.284496736f);
    p = __builtin_fmaf(p, t, 0.5f * 0.254829592f);
    p *= t;
    e = __expf(-ax * ax);
    return copysignf(__builtin_fmaf(-p, e, 0.5f), x);
}

// GELU(z) = z Phi(z) = z (1/2 + erf(z / sqrt 2) / 2) and its derivative
// Phi(z) + z phi(z), phi(z) = exp(-z^2 / 2) / sqrt(2 pi).
__device__ __forceinline__ float gelu(float z)
{
    float e;
    return z * (0.5f + half_erf(z * 0.70710678118654752f, e));
}
__device__ __forceinline__ float gelu_grad(float z)
{
    float e;
    const float er = half_erf(z * 0.70710678118654752f, e);
    return (0.5f + er) + z * e * 0.39894228040143268f;
}

__device__ __forceinline__ int wrapc(int i, int n) { return i < 0 ? i + n : (i >= n ? i - n : i); }

__device__ __forceinline__ bf16x8 load8(const u16 *p)
{
    const uint4 q = *reinterpret_cast<const uint4 *>(p);
    return __builtin_bit_cast(bf16x8, q);
}

__device__ __forceinline__ uint4 pack8(const u16 (&v)[8])
{
    return uint4{(uint32_t)v[0] | ((uint32_t)v[1] << 16), (uint32_t)v[2] | ((uint32_t)v[3] << 16),
                 (uint32_t)v[4] | ((uint32_t)v[5] << 16), (uint32_t)v[6] | ((uint32_t)v[7] << 16)};
}

// Workgroup barrier that waits for the wave's LDS operations only: global
// loads in flight (the next planes' staging) stay in flight across it.
__device__ __forceinline__ void wg_lds_barrier()
{
    __builtin_amdgcn_s_waitcnt(0xC07F); // lgkmcnt(0); vmcnt and expcnt not waited
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    __builtin_amdgcn_s_barrier();
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
}

// ------------------------------------------------------------------ convolution
// MODE_HIDDEN: z = acc + bias, writes z and GELU(z) (32 channels, BF16).
// MODE_ACT:    the same, writing GELU(z) only (inference keeps no z).
// MODE_OUT:    pred = residual input + acc + bias for output channels 0, 1.
// MODE_DGRAD:  writes acc * GELU'(zprev) (the gradient of the layer below's
//              pre-activation, 32 channels, BF16).
template <int N> struct IntC {
    static constexpr int value = N;
};
constexpr int PX = 16;      // cells of a patch in x
constexpr int RX = PX + 2;  // with the ring around it

// 8 -> 32 convolutions (the first layer, and the data gradient of the last): as
// conv32p_kernel below, a wavefront owns RW rows of 16 cells and both 16-channel N
// tiles of one sample and marches through a chunk of z planes with a private LDS
// ring, here of the three planes that a K chunk (four neighbour cells) may reach
// into; no barriers. All 14 weight fragments sit in registers. The two tiles'
// output channels are interleaved so that a lane holds 8 consecutive channels and a
// wavefront stores (and the data gradient reads) whole 1 KB rows in 16-byte
// accesses. Loads run a plane ahead; the chunk's planes are a multiple of three, the
// ring's phases.
// What bounds it: the stores of a hidden layer's two tensors (1.07 GB at 4 x 128^3,
// 3.4 TB/s), the data gradient's 1.2 GB (the rate of a large copy), and for a
// prediction the GELU's 16 vector operations a value. With workgroups sharing a ring
// behind two barriers a plane, and the weights in LDS: forward 346 -> 320 us, data
// gradient 302 -> 238, one prediction's layer at 128^3 74 -> 65. Four rows a
// wavefront, or four wavefronts a SIMD, are no faster.
constexpr int C8_RW = 2, C8_WAVES = 4;
template <int MODE>
__global__ __launch_bounds__(64 * C8_WAVES) __attribute__((amdgpu_waves_per_eu(3, 3))) void conv8_kernel(ConvArgs a)
{
    constexpr int NT = 2, NCH = 7, RW = C8_RW, PYW = RW * C8_WAVES;
    constexpr int RCELLS = RX * (RW + 2);             // ring cells per plane, a 16-byte vector each
    constexpr int SLOT_V = (RCELLS + 15) / 16 * 16;
    constexpr int LOADS = (RCELLS + 63) / 64;
    // behind the rings RW rows of zeros: the last chunk has 27 - 24 = 3 cells
    constexpr int ZERO = C8_WAVES * 3 * SLOT_V;
    __shared__ u32x4 ring_all[ZERO + (RW - 1) * RX + 1];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int col = lane & 15, quad = lane >> 4;
    const Geo g = a.geo;
    const int ring0 = wave * 3 * SLOT_V;

    bf16x8 w[NCH][NT];
#pragma unroll
    for (int c = 0; c < NCH; ++c)
#pragma unroll
        for (int t = 0; t < NT; ++t) w[c][t] = load8(a.wpack + ((c * NT + t) * 64 + lane) * 8);
    if ((int)threadIdx.x < (RW - 1) * RX + 1) ring_all[ZERO + threadIdx.x] = u32x4{0u, 0u, 0u, 0u};
    __syncthreads();

    const int tx = g.nx / PX, ty = (g.ny + PYW - 1) / PYW, tzc = (g.nz + a.zc - 1) / a.zc;
    int b = blockIdx.x;
    const int bx = b % tx;
    b /= tx;
    const int by = b % ty;
    b /= ty;
    const int bz = b % tzc;
    const int s = b / tzc;
    const int x0 = bx * PX, yw = by * PYW + RW * wave, z0 = min(bz * a.zc, g.nz - a.zc), ze = z0 + a.zc;
    if (yw >= g.ny) return; // a wavefront below the grid (no barriers after this point)
    const size_t sbase = (size_t)s * g.ncell, plane = (size_t)g.nx * g.ny;

    // This lane's ring vectors (cells; lanes past the plane repeat the last one).
    uint32_t goff[LOADS];
    int rpos[LOADS];
#pragma unroll
    for (int l = 0; l < LOADS; ++l) {
        rpos[l] = min(lane + 64 * l, RCELLS - 1);
        int gy = yw + rpos[l] / RX - 1;
        if (gy < 0) gy += g.ny;
        while (gy >= g.ny) gy -= g.ny;
        goff[l] = (uint32_t)wrapc(x0 + rpos[l] % RX - 1, g.nx) + (uint32_t)g.nx * gy;
    }
    auto load_plane = [&](int z, u32x4 (&o)[LOADS]) __attribute__((always_inline)) {
        const u32x4 *base = reinterpret_cast<const u32x4 *>(a.in) + sbase + (size_t)wrapc(z, g.nz) * plane;
#pragma unroll
        for (int l = 0; l < LOADS; ++l) o[l] = base[goff[l]];
    };
    auto stage_plane = [&](int slot, const u32x4 (&o)[LOADS]) __attribute__((always_inline)) {
#pragma unroll
        for (int l = 0; l < LOADS; ++l) ring_all[ring0 + slot * SLOT_V + rpos[l]] = o[l];
    };
    // Chunk c's cell of this lane (offset 4 c + quad) in phase P, where plane z + dz - 1
    // sits in slot (P + dz) mod 3.
    int at0[NCH], at1[NCH], at2[NCH];
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
        const int d = 4 * c + quad, cell = ring0 + d / 3 % 3 * RX + d % 3 + col;
        at0[c] = d < 27 ? cell + d / 9 * SLOT_V : ZERO;
        at1[c] = d < 27 ? cell + (d / 9 + 1) % 3 * SLOT_V : ZERO;
        at2[c] = d < 27 ? cell + (d / 9 + 2) % 3 * SLOT_V : ZERO;
    }
    float bias_r[8] = {};
    if constexpr (MODE != MODE_DGRAD) {
#pragma unroll
        for (int c = 0; c < 8; ++c) bias_r[c] = a.bias[8 * quad + c];
    }
    const uint32_t lane_c = col * 32 + quad * 8;
    auto out_at = [&](int r, int z) __attribute__((always_inline)) {
        return (sbase + (size_t)x0 + (size_t)g.nx * ((size_t)min(yw + r, g.ny - 1) + (size_t)g.ny * z)) * 32;
    };
    bf16x8 zq[RW] = {}; // MODE_DGRAD: this plane's pre-activations
    auto load_zq = [&](int r, int z) __attribute__((always_inline)) {
        if constexpr (MODE == MODE_DGRAD) zq[r] = load8(a.zprev + out_at(r, z) + lane_c);
    };
    auto step = [&](auto phase, int z) __attribute__((always_inline)) {
        constexpr int P = decltype(phase)::value;
        u32x4 pre[LOADS];
        load_plane(z + 2, pre);
        f32x4 acc[RW][NT];
#pragma unroll
        for (int r = 0; r < RW; ++r)
#pragma unroll
            for (int t = 0; t < NT; ++t) acc[r][t] = f32x4{0.f, 0.f, 0.f, 0.f};
        constexpr int KD = 2; // fragments are read KD chunks ahead of their MFMAs
        bf16x8 av[KD][RW];
        auto frag = [&](int c) __attribute__((always_inline)) {
#pragma unroll
            for (int r = 0; r < RW; ++r) av[c % KD][r] = __builtin_bit_cast(bf16x8, ring_all[(P == 0 ? at0[c] : P == 1 ? at1[c] : at2[c]) + r * RX]);
        };
#pragma unroll
        for (int c = 0; c < KD; ++c) frag(c);
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
#pragma unroll
            for (int r = 0; r < RW; ++r)
#pragma unroll
                for (int t = 0; t < NT; ++t)
                    acc[r][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[c][t], av[c % KD][r], acc[r][t], 0, 0, 0);
            if (c + KD < NCH) frag(c + KD);
            __builtin_amdgcn_sched_barrier(0);
        }
        // acc[r][t][j]: output channel 8 quad + 4 t + j of cell (x0 + col, yw + r, z).
        u16 e1[RW][8], e2[RW][8];
#pragma unroll
        for (int r = 0; r < RW; ++r) {
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                const float v = acc[r][c / 4][c % 4];
                if constexpr (MODE == MODE_DGRAD) {
                    e1[r][c] = f2bf(v * gelu_grad((float)zq[r][c]));
                } else {
                    const float zz = v + bias_r[c];
                    e1[r][c] = f2bf(MODE == MODE_HIDDEN ? zz : gelu(zz));
                    if constexpr (MODE == MODE_HIDDEN) e2[r][c] = f2bf(gelu(zz));
                }
            }
            load_zq(r, min(z + 1, ze - 1));
        }
        stage_plane((P + 3) % 3, pre); // plane z + 2 replaces z - 1
        // rows last to first: a row past the grid (only when ny is odd) is
        // clamped onto row 0's cell, whose own store then follows it
#pragma unroll
        for (int r = RW - 1; r >= 0; --r) {
            const size_t o = out_at(r, z);
            *reinterpret_cast<uint4 *>((MODE == MODE_HIDDEN ? a.zout : a.aout) + o + lane_c) = pack8(e1[r]);
            if constexpr (MODE == MODE_HIDDEN) *reinterpret_cast<uint4 *>(a.aout + o + lane_c) = pack8(e2[r]);
        }
    };
#pragma unroll
    for (int p = 0; p < 3; ++p) {
        u32x4 q[LOADS];
        load_plane(z0 - 1 + p, q);
        stage_plane(p, q);
    }
#pragma unroll
    for (int r = 0; r < RW; ++r) load_zq(r, z0);
    for (int z = z0; z < ze; z += 3) {
        step(IntC<0>{}, z);
        step(IntC<1>{}, z + 1);
        step(IntC<2>{}, z + 2);
    }
}

// Output layer (32 -> 2 channels, residual added). As an implicit GEMM over the
// 27 offsets its 2 output channels fill 2 of an MFMA tile's 16 rows. Here the
// rows are the 9 (y, x) offsets of both channels instead (18 rows, two tiles),
// and K runs over the 32 channels and the three z offsets:
//   Q[dy, dx, o](x, y, z) = sum over dz, c of W[o][c][dz, dy, dx] a(x, y, z + dz, c),
//   out[o](x, y, z) = sum over dy, dx of Q[dy, dx, o](x + dx, y + dy, z),
// six MFMAs per 16 cells instead of 27 and every activation fragment read once,
// straight from memory (16 cells x 64 bytes are contiguous). The nine shifted
// terms of an output are added from LDS, 144 bytes of traffic per cell instead
// of 1.7 KB of fragments.
//
// A workgroup of eight wavefronts owns OUT_TY output rows of up to OUT_NG
// 16-cell groups (a whole row when it fits, else OUT_NG - 2 output groups
// between two halo groups) of one sample and marches through a chunk of z
// planes; wavefront w computes Q of region row y0 - 1 + w. Planes z - 1, z and
// z + 1 sit in registers (five slots, planes z + 2 and z + 3 on their way), Q in
// one of two LDS buffers, so there is one barrier per plane, which waits for LDS
// operations only.
// What bounds it: the read of the activations (0.54 GB at 4 x 128^3, 0.11 ms at
// the rate of a large copy; a third more with the rows two workgroups read).
// 4 x 128^3: 176 us (363 as an implicit GEMM over 27 offsets). The prefetch has
// to stay in flight: waits are in order, so with the residual inputs loaded
// after it, or the addresses in spilled registers, a plane cost 250 us' worth of
// exposed latency.
constexpr int OUT_TY = 6, OUT_NG = 8, OUT_COLS = 16 * OUT_NG;
constexpr int OUT_PLANE = (OUT_TY + 2) * OUT_COLS + 8; // float2 per (dy, dx); the pad spreads the quads' writes over the banks
// FULL: rows of at least OUT_NG groups, so that every load is unconditional (the
// compiler's waits then count the loads in flight; behind conditions they drain
// them).
template <typename IO, bool FULL>
__global__ __launch_bounds__(512) void conv_out_kernel(ConvArgs a)
{
    __shared__ float2 q_l[2][9 * OUT_PLANE];
    const Geo g = a.geo;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int col = lane & 15, quad = lane >> 4;
    const int ng = g.nx / 16;
    const bool whole = ng <= OUT_NG;                // the tile is the whole row (periodic in itself)
    const int tg = whole ? ng : OUT_NG - 2;         // output groups of a tile
    const int rg = whole ? ng : OUT_NG;             // groups computed
    const int tx = (ng + tg - 1) / tg, ty = (g.ny + OUT_TY - 1) / OUT_TY, tzc = (g.nz + a.zc - 1) / a.zc;
    int b = blockIdx.x;
    const int bx = b % tx;
    b /= tx;
    const int by = b % ty;
    b /= ty;
    const int bz = b % tzc;
    const int s = b / tzc;
    const int g0 = bx * tg, y0 = by * OUT_TY, z0 = bz * a.zc, ze = min(z0 + a.zc, g.nz);
    const size_t sbase = (size_t)s * g.ncell, plane = (size_t)g.nx * g.ny;

    bf16x8 w[3][2];
#pragma unroll
    for (int d = 0; d < 3; ++d)
#pragma unroll
        for (int t = 0; t < 2; ++t) w[d][t] = load8(a.wpack + ((d * 2 + t) * 64 + lane) * 8);

    // Every address is a wavefront's base plus this lane's bytes. Group i of
    // region row `wave` starts at cell row + gcell[i] of a plane; a lane reads 8
    // channels of its cell.
    const size_t row = sbase + (size_t)((y0 - 1 + wave + g.ny) % g.ny) * g.nx;
    int gcell[OUT_NG];
#pragma unroll
    for (int i = 0; i < OUT_NG; ++i) gcell[i] = 16 * ((g0 + (whole ? min(i, ng - 1) : i - 1) + ng) % ng);
    const uint32_t lane_b = col * 64 + quad * 16;
    bf16x8 f[5][OUT_NG]; // plane z in slot (z - z0 + 1) mod 5
    auto load_plane = [&](int z, bf16x8 (&o)[OUT_NG]) __attribute__((always_inline)) {
        const u16 *base = a.in + (row + (size_t)wrapc(z, g.nz) * plane) * 32;
#pragma unroll
        for (int i = 0; i < OUT_NG; ++i)
            if (FULL || i < rg)
                o[i] = load8(reinterpret_cast<const u16 *>(reinterpret_cast<const char *>(base + (size_t)gcell[i] * 32) + lane_b));
    };
    const float2 bias = {a.bias[0], a.bias[1]};
    // This lane's outputs: column x of rows wave / 2 and 4 more.
    const int xw = (wave & 1) * 64, x = xw + lane, row0 = wave >> 1;
    const int c = (whole ? 0 : 16) + x; // its column in the region
    const int cl = whole && c == 0 ? g.nx - 1 : c - 1, cr = whole && c == g.nx - 1 ? 0 : c + 1;
    const int ncol = min(16 * tg, g.nx - 16 * g0);
    const bool x_ok = x < ncol;
    bool row_ok[2];
    size_t out_row[2]; // (rows without outputs load a valid residual, as do lanes past the tile)
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        row_ok[h] = row0 + 4 * h < OUT_TY && y0 + row0 + 4 * h < g.ny;
        out_row[h] = sbase + (row_ok[h] ? (size_t)(y0 + row0 + 4 * h) * g.nx + 16 * g0 : 0);
    }
    const uint32_t out_b = (uint32_t)min(x, ncol - 1) * (uint32_t)sizeof(IO);
    auto io_at = [&](const void *p, size_t e) __attribute__((always_inline)) {
        return reinterpret_cast<IO *>(const_cast<char *>(static_cast<const char *>(p)) + e * sizeof(IO) + out_b);
    };
    auto step = [&](int z, auto phase) __attribute__((always_inline)) {
        constexpr int P = decltype(phase)::value; // (z - z0) mod 5
        // The residual inputs are loaded before the prefetch: loads complete in
        // order, and waiting for them must not wait for it.
        IO res[2][2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const size_t r = out_row[h] + (size_t)z * plane;
            res[h][0] = *io_at(a.res_u, r);
            res[h][1] = *io_at(a.res_v, r);
        }
        __builtin_amdgcn_sched_barrier(0);
        load_plane(min(z + 3, ze), f[(P + 4) % 5]);
        float2 *q = q_l[(z - z0) & 1];
#pragma unroll
        for (int i = 0; i < OUT_NG; ++i) {
            if (!FULL && i >= rg) break;
            f32x4 acc[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
            for (int d = 0; d < 3; ++d)
#pragma unroll
                for (int t = 0; t < 2; ++t)
                    acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[d][t], f[(P + d) % 5][i], acc[t], 0, 0, 0);
            // acc[t][j]: row 16 t + 4 quad + j = 2 (3 dy + dx) + o of cell (16 i + col)
            float2 *dst = q + wave * OUT_COLS + 16 * i + col;
            dst[(2 * quad) * OUT_PLANE] = float2{acc[0][0], acc[0][1]};
            dst[(2 * quad + 1) * OUT_PLANE] = float2{acc[0][2], acc[0][3]};
            if (quad == 0) dst[8 * OUT_PLANE] = float2{acc[1][0], acc[1][1]};
            if (i & 1) __builtin_amdgcn_sched_barrier(0);
        }
        wg_lds_barrier();
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            if (!(row_ok[h] && x_ok)) continue;
            float2 sum = bias;
#pragma unroll
            for (int dy = 0; dy < 3; ++dy) {
                const float2 *p = q + 3 * dy * OUT_PLANE + (row0 + 4 * h + dy) * OUT_COLS;
                const float2 l = p[cl], m = p[OUT_PLANE + c], r = p[2 * OUT_PLANE + cr];
                sum.x += (l.x + m.x) + r.x;
                sum.y += (l.y + m.y) + r.y;
            }
            const size_t r = out_row[h] + (size_t)z * plane;
            *io_at(a.out_u, r) = res[h][0] + (IO)sum.x;
            *io_at(a.out_v, r) = res[h][1] + (IO)sum.y;
        }
    };
#pragma unroll
    for (int p = 0; p < 4; ++p) load_plane(z0 - 1 + p, f[p]);
    for (int z = z0; z < ze; z += 5) {
        step(z, IntC<0>{});
        if (z + 1 < ze) step(z + 1, IntC<1>{});
        if (z + 2 < ze) step(z + 2, IntC<2>{});
        if (z + 3 < ze) step(z + 3, IntC<3>{});
        if (z + 4 < ze) step(z + 4, IntC<4>{});
    }
}
// 32 -> 32 convolutions of the forward hidden layer (with or without the
// pre-activation's store) and the data gradient. A wavefront owns RW rows of
// 16 cells and both 16-channel N tiles of one sample and marches through a chunk
// of z planes. Input plane p adds to the outputs of planes p + 1, p and p - 1 (z
// offsets -1, 0, +1), which sit in three sets of accumulators, so an activation
// fragment is read from LDS once for all z offsets and for the rows it is a
// neighbour of: 12 reads per plane where a loop over the 27 offsets takes 54. The
// plane in work and the next one sit in a private LDS ring (rows y-1 .. y+RW, cells
// x-1 .. x+16, channel group major, groups C32_GC cells apart so that the staging
// writes of a cell's four groups meet different banks), so the wavefronts of a
// workgroup meet at one barrier only, after the weights are staged. Every ninth K
// chunk's weight fragments sit in registers and the others' in LDS (shared by the
// workgroup's eight wavefronts), which leaves room for two wavefronts per SIMD: one
// wavefront's vector work (the epilogue, the staging) then runs beside the
// other's MFMAs. Plane p's MFMAs and the epilogue (bias, GELU or its derivative,
// BF16 rounding) of the plane finished before sit in one basic block, in four
// copies, as the finished set and the three in work rotate. Each output still adds
// its 27 K chunks in the order z, y, x: the results are those of a loop over the
// offsets, bit for bit.
// What bounds it: power. MFMAs alone on random data run at 1.7 GHz and 1730
// TFLOP/s, with six vector instructions per 32 clocks of MFMA at 1265 to 1335; this
// kernel reaches 1070 (forward) and 980 (data gradient). At 4 x 128^3 the loop over
// the offsets took 450 and 500 us, with 65% of its cycles spent on LDS reads, and
// this one 435 and 470; one prediction's layer at 128^3 140 -> 116 us (the pre-
// activations are then not stored: 1.07 of 1.6 GB). More weights in registers, other
// read distances and group strides make no difference any more.
constexpr int C32_RW = 2, C32_WAVES = 8, C32_EVERY = 9;
template <bool B> struct BoolC {
    static constexpr bool value = B;
};
// One step of the march: the z offsets LO .. LO + NZ - 1 (of 0, 1, 2) that add,
// whether a finished plane has its epilogue, and whether another plane follows.
// Group k of a step works on chunk (3 dy + dx) 3 + dz.
template <int PHASE_, int LO_, int NZ_, bool PREV_, bool MORE_> struct C32Step {
    static constexpr int PHASE = PHASE_, LO = LO_, NZ = NZ_;
    static constexpr bool PREV = PREV_, MORE = MORE_;
    static constexpr int chunk(int k) { return k / NZ * 3 + LO + k % NZ; }
};
template <int MODE>
__global__ __launch_bounds__(64 * C32_WAVES) __attribute__((amdgpu_waves_per_eu(2, 2))) void conv32p_kernel(ConvArgs a)
{
    constexpr int NT = 2, NCH = 27, VPC = 4, RW = C32_RW, PYW = RW * C32_WAVES, EV = C32_EVERY;
    constexpr int RCELLS = RX * (RW + 2);              // ring cells per plane
    constexpr int GC = RCELLS + 12;                    // cells per channel group: 5.25 times 256 bytes
    constexpr int SLOT_V = GC * VPC;                   // 16-byte vectors per plane slot
    constexpr int LOAD_V = RCELLS * VPC;               // vectors loaded per plane
    constexpr int LOADS = (LOAD_V + 63) / 64;
    constexpr int CR = (NCH + EV - 1) / EV, CL = NCH - CR; // weight chunks in registers / in LDS
    __shared__ u32x4 ring_all[C32_WAVES * 2 * SLOT_V];
    __shared__ uint4 wl[CL * NT * 64];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    u32x4 *ring = ring_all + wave * 2 * SLOT_V;
    const int col = lane & 15, quad = lane >> 4;
    const Geo g = a.geo;

    // Chunk i = (3 dy + dx) 3 + dz; the packed weights are in the order 9 dz + 3 dy + dx.
    auto packed = [](int i) { return i % 3 * 9 + i / 3; };
    bf16x8 wr[CR][NT];
    {
        const uint4 *wg = reinterpret_cast<const uint4 *>(a.wpack);
#pragma unroll
        for (int c = 0; c < CR; ++c)
#pragma unroll
            for (int t = 0; t < NT; ++t) wr[c][t] = __builtin_bit_cast(bf16x8, wg[(packed(c * EV) * NT + t) * 64 + lane]);
        for (int e = threadIdx.x; e < CL * NT * 64; e += 64 * C32_WAVES) {
            const int l = e / (NT * 64), i = l / (EV - 1) * EV + l % (EV - 1) + 1; // the l-th chunk that is no multiple of EV
            wl[e] = wg[packed(i) * NT * 64 + e % (NT * 64)];
        }
    }
    __syncthreads();
    const int tx = g.nx / PX, ty = (g.ny + PYW - 1) / PYW, tzc = (g.nz + a.zc - 1) / a.zc;
    int b = blockIdx.x;
    const int bx = b % tx;
    b /= tx;
    const int by = b % ty;
    b /= ty;
    const int bz = b % tzc;
    const int s = b / tzc;
    const int x0 = bx * PX, yw = by * PYW + RW * wave, z0 = min(bz * a.zc, g.nz - a.zc), ze = z0 + a.zc;
    if (yw >= g.ny) return; // a wavefront below the grid (no barriers after this point)
    const size_t sbase = (size_t)s * g.ncell, plane = (size_t)g.nx * g.ny;

    // This lane's ring vectors: offset within an input plane (in vectors)
    // and ring position; the lanes past the plane load a valid vector and
    // store it into padding.
    uint32_t goff[LOADS];
    int rpos[LOADS];
#pragma unroll
    for (int l = 0; l < LOADS; ++l) {
        const int v = min(lane + 64 * l, LOAD_V - 1);
        const int cell = v / VPC, cg = v % VPC;
        const int rx = cell % RX, ry = cell / RX;
        int gy = yw + ry - 1;
        if (gy < 0) gy += g.ny;
        while (gy >= g.ny) gy -= g.ny;
        const int gx = wrapc(x0 + rx - 1, g.nx);
        goff[l] = ((uint32_t)gx + (uint32_t)g.nx * gy) * VPC + cg; // at most 4 x 2.5e8
        rpos[l] = lane + 64 * l < LOAD_V ? cg * GC + cell : 3 * GC + RCELLS + (lane & 7);
    }
    auto load_plane = [&](int z, u32x4 (&o)[LOADS]) __attribute__((always_inline)) {
        const u32x4 *base = reinterpret_cast<const u32x4 *>(a.in + (sbase + (size_t)wrapc(z, g.nz) * plane) * 32);
#pragma unroll
        for (int l = 0; l < LOADS; ++l) o[l] = base[goff[l]];
    };
    // Epilogue values: the lane's biases are read once (the compiler cannot
    // move their loads past the output stores).
    float bias_r[NT][4] = {};
    if constexpr (MODE == MODE_HIDDEN || MODE == MODE_ACT) {
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int j = 0; j < 4; ++j) bias_r[t][j] = a.bias[8 * quad + 4 * t + j];
    }
    // This lane's 8 channels of its cell of row r, plane z: a wavefront's base and
    // the lane's offset.
    const uint32_t lane_c = col * 32 + quad * 8;
    auto out_at = [&](int r, int z) __attribute__((always_inline)) {
        return (sbase + (size_t)x0 + (size_t)g.nx * ((size_t)min(yw + r, g.ny - 1) + (size_t)g.ny * z)) * 32;
    };
    bf16x8 zq[RW] = {};  // MODE_DGRAD: pre-activations of the plane whose epilogue is next
    f32x4 acc[4][RW][NT]; // output plane z in set (z - z0 + 1) mod 4
    u16 e1[RW][8], e2[RW][8]; // 8 consecutive channels per lane and row
    auto value = [&](int v, const f32x4 (&f)[RW][NT]) __attribute__((always_inline)) {
        const int r = v / (NT * 4), t = (v / 4) % NT, j = v % 4;
        // the empty asm keeps each value's arithmetic where it stands
        // (pure arithmetic would otherwise sink to the stores)
        if constexpr (MODE == MODE_HIDDEN) {
            float zz = f[r][t][j] + bias_r[t][j];
            float gz = gelu(zz);
            asm volatile("" : "+v"(zz), "+v"(gz));
            e1[r][4 * t + j] = f2bf(zz);
            e2[r][4 * t + j] = f2bf(gz);
        } else if constexpr (MODE == MODE_ACT) {
            float gz = gelu(f[r][t][j] + bias_r[t][j]);
            asm volatile("" : "+v"(gz));
            e1[r][4 * t + j] = f2bf(gz);
        } else {
            float gd = f[r][t][j] * gelu_grad((float)zq[r][4 * t + j]);
            asm volatile("" : "+v"(gd));
            e1[r][4 * t + j] = f2bf(gd);
        }
    };
    auto store_plane = [&](int z) __attribute__((always_inline)) {
        // rows last to first: a row past the grid (only when ny is odd) is
        // clamped onto row 0's cell, whose own store then follows it
#pragma unroll
        for (int r = RW - 1; r >= 0; --r) {
            const size_t o = out_at(r, z);
            *reinterpret_cast<uint4 *>((MODE == MODE_HIDDEN ? a.zout : a.aout) + o + lane_c) = pack8(e1[r]);
            if constexpr (MODE == MODE_HIDDEN) *reinterpret_cast<uint4 *>(a.aout + o + lane_c) = pack8(e2[r]);
        }
    };
    // Input plane p (in slot PHASE mod 2, PHASE = p - z0 + 1 mod 4): start loading
    // plane p + 1, run the K chunks with the 16 epilogue values of plane p - 2 (2
    // rows x 2 tiles x 4 channels) spread over them, then stage plane p + 1 and
    // store plane p - 2.
    auto step = [&](auto kind, int p) __attribute__((always_inline)) {
        typedef decltype(kind) K;
        constexpr int P = K::PHASE, NG = 9 * K::NZ, NV = RW * NT * 4, KD = 3;
        u32x4 pre[LOADS];
        if constexpr (K::MORE) load_plane(p + 1, pre);
        const f32x4 (&fin)[RW][NT] = acc[(P + 2) % 4]; // plane p - 2
#pragma unroll
        for (int r = 0; r < RW; ++r)
#pragma unroll
            for (int t = 0; t < NT; ++t) acc[(P + 1) % 4][r][t] = f32x4{0.f, 0.f, 0.f, 0.f};
        const u32x4 *rs = ring + P % 2 * SLOT_V + quad * GC + col;
        bf16x8 av[3][3], wv[KD][NT]; // ring row R in av[R % 3]
        auto read_row = [&](int R, int dx) __attribute__((always_inline)) {
            av[R % 3][dx] = __builtin_bit_cast(bf16x8, rs[R * RX + dx]);
        };
        auto read_w = [&](int k) __attribute__((always_inline)) {
            const int i = K::chunk(k);
            if (i % EV != 0) {
#pragma unroll
                for (int t = 0; t < NT; ++t)
                    wv[k % KD][t] = __builtin_bit_cast(bf16x8, wl[((i - i / EV - 1) * NT + t) * 64 + lane]);
            }
        };
        read_row(0, 0);
        read_row(1, 0);
        read_w(0);
        read_row(0, 1);
        read_row(1, 1);
        read_w(1);
        read_row(0, 2);
        read_row(1, 2);
        read_w(2);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int k = 0; k < NG; ++k) {
            const int i = K::chunk(k), dz = i % 3, dx = i / 3 % 3, dy = i / 9;
            f32x4 (&o)[RW][NT] = acc[(P + 5 - dz) % 4]; // plane p + 1 - dz
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int r = 0; r < RW; ++r)
                    o[r][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(i % EV == 0 ? wr[i / EV][t] : wv[k % KD][t],
                                                                      av[(dy + r) % 3][dx], o[r][t], 0, 0, 0);
            if (k + KD < NG) read_w(k + KD);
            // row dy + 2 replaces row dy - 1, from the second offset's groups on
            if (dy < 2 && k % K::NZ == 0) read_row(dy + 2, dx);
            if constexpr (K::PREV) {
#pragma unroll
                for (int v = k * NV / NG; v < (k + 1) * NV / NG; ++v) value(v, fin);
            }
            if constexpr (MODE == MODE_DGRAD && K::LO + K::NZ == 3) {
#pragma unroll
                for (int r = 0; r < RW; ++r) // row r's values are done: its next plane's
                    if ((k + 1) * NV / NG >= (r + 1) * NT * 4 && k * NV / NG < (r + 1) * NT * 4)
                        zq[r] = load8(a.zprev + out_at(r, p - 1) + lane_c);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (K::MORE) {
            u32x4 *dst = ring + (P + 1) % 2 * SLOT_V;
#pragma unroll
            for (int l = 0; l < LOADS; ++l) dst[rpos[l]] = pre[l];
        }
        if constexpr (K::PREV) store_plane(p - 2);
    };
    {
        u32x4 q[LOADS];
        load_plane(z0 - 1, q);
#pragma unroll
        for (int l = 0; l < LOADS; ++l) ring[rpos[l]] = q[l];
    }
    step(C32Step<0, 0, 1, false, true>{}, z0 - 1);
    step(C32Step<1, 0, 2, false, true>{}, z0);
    step(C32Step<2, 0, 3, false, true>{}, z0 + 1);
    step(C32Step<3, 0, 3, true, true>{}, z0 + 2);
    int p = z0 + 3;
    for (; p + 1 < ze; p += 4) {
        step(C32Step<0, 0, 3, true, true>{}, p);
        step(C32Step<1, 0, 3, true, true>{}, p + 1);
        step(C32Step<2, 0, 3, true, true>{}, p + 2);
        step(C32Step<3, 0, 3, true, true>{}, p + 3);
    }
    step(C32Step<0, 1, 2, true, true>{}, p);
    step(C32Step<1, 2, 1, true, false>{}, p + 1);
#pragma unroll
    for (int v = 0; v < RW * NT * 4; ++v) value(v, acc[0]);
    store_plane(p);
}
// ------------------------------------------------------------------ weight gradient
// dW[d][co][ci] = sum over cells of dz[cell][co] * act[cell + d][ci]: for each
// of the 27 offsets d a product A B with A = dz^T (rows co, K = cells) and
// B = act shifted by d (K = cells, columns ci), on 16x16x32 MFMAs whose K runs
// over 32 cells (two rows of 16).
//
// The workgroups are persistent: each walks work items (a patch of 16 x-cells
// by TR = 8 y-rows of one sample, through a chunk of WG_ZC planes; 8 rows load 10
// activation rows per 8 where 4 would load 6 per 4) and keeps its sums in
// registers. Act plane p meets dz planes p + 1, p and p - 1 (z offsets -1, 0,
// +1), so the loop runs over act planes: while plane p is in LDS, the dz
// fragments of the three planes it meets are held in registers, and every B
// fragment read from LDS feeds three MFMAs, one per z offset (a third of the LDS
// reads of a loop that takes the offsets one by one). For each offset the planes
// are still added in increasing z. Both operands stay channels-last in LDS, as in
// memory (16-byte chunks, no transposes on the way in): a fragment (8 cells of
// one channel per lane) is two transposing LDS reads. Cells 8 .. 15 of every 16
// have their channel halves swapped, so that the two 16-lane groups of a
// half-wave read distinct banks.
//
// Wave w owns one 16 x 16 output tile (co x ci) for all 27 offsets and all K
// chunks of a plane (two rows of 16 cells each). Act plane p + 2 and dz plane p + 3
// are stored into the third of three LDS slots half way through plane p, behind the
// plane's one barrier, and loaded a step before; the B fragments are read a few
// MFMAs ahead across the planes, so no wavefront starts a plane waiting for LDS or
// for the others. The bias gradient (the sum of dz over cells) is accumulated while
// dz is staged. Each workgroup writes its partial sums (32 x 32 per offset, and 32
// bias sums) once.
// What bounds it: the matrix units at the clock that the card's power allows (1300
// TFLOP/s; MFMAs with their LDS reads alone 1540 to 1660). 4 x 128^3: 452 -> 355 us
// against two slots with the barrier between planes and the staged vectors as
// structs, which the compiler kept in LDS, waiting for each load where it was issued.
constexpr int WG_ZC = 64;

typedef short v4s __attribute__((ext_vector_type(4)));

// Offset (16-bit units) of channel ch of cell `cell` in an LDS row of
// channels-last cells of 32 channels, with the bank swizzle described above.
__device__ __forceinline__ int wg_pos(int cell, int ch) { return cell * 32 + (ch ^ ((cell & 8) << 1)); }

// MFMA operand of cells cell0 .. cell0 + 7 and channels c0 .. c0 + 15 (one per
// lane of a 16-lane group) from an LDS row. In each group of 16 lanes the
// transposing read concatenates the 8-byte pieces the lanes address, in lane
// order, into 64 values X and hands lane t the values X[t], X[t + 16],
// X[t + 32] and X[t + 48]; so lane L addresses cell L / 4 (then 4 + L / 4)
// at channels c0 + 4 (L % 4) .. + 3, and receives channel c0 + L of the
// 8 cells.
__device__ __forceinline__ bf16x8 frag_tr(const u16 *row, int cell0, int c0, int lane16)
{
    const int cell = cell0 + (lane16 >> 2), ch = c0 + 4 * (lane16 & 3);
    typedef __attribute__((address_space(3))) v4s *lds_v4s;
    const v4s lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s)(row + wg_pos(cell, ch)));
    const v4s hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s)(row + wg_pos(cell + 4, ch)));
    const v4s v[2] = {lo, hi};
    return __builtin_bit_cast(bf16x8, v);
}

__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void wgrad_kernel(WgradArgs a)
{
    constexpr int CIN = 32, COUTS = 32, MT = 2, NT = 2, TR = 8;
    constexpr int NCI = 16 * NT, NCO = 16 * MT;
    constexpr int NCG = CIN / 8, NCGZ = COUTS / 8;
    constexpr int NKC = TR / 2;              // K chunks (two rows of 16 cells) per wave and plane
    constexpr int AROW = (18 * NCI * 2 + 255) / 256 * 256 / 2; // u16 per act row: cells x0 - 1 .. x0 + 16
    constexpr int APL = (TR + 2) * AROW;                        // act rows y0 - 1 .. y0 + TR
    constexpr int DROW = 16 * NCO, DPL = TR * DROW;             // dz rows y0 .. y0 + TR - 1
    constexpr int T_ACT = (TR + 2) * 18 * NCG, RA = (T_ACT + 255) / 256; // 16-byte chunks of an act plane
    constexpr int T_DZ = TR * 16 * NCGZ;                                  // and of a dz plane
    constexpr int RD = T_DZ / 256;              // dz chunks per lane
    static_assert(T_DZ % 256 == 0, "whole dz rounds");
    __shared__ __align__(16) u16 act_l[3 * APL];
    __shared__ __align__(16) u16 dz_l[3 * DPL];
    __shared__ float bsum_l[256][8];
    const Geo g = a.geo;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int col = lane & 15, quad = lane >> 4;
    const int mw = wave >> 1, nw = wave & 1; // the wave's output tile


    f32x4 acc[27];
#pragma unroll
    for (int d = 0; d < 27; ++d) acc[d] = f32x4{0.f, 0.f, 0.f, 0.f};
    float bs[8];
#pragma unroll
    for (int c = 0; c < 8; ++c) bs[c] = 0.f;

    const int ntx = g.nx / 16, nty = (g.ny + TR - 1) / TR, ntz = (g.nz + WG_ZC - 1) / WG_ZC;
    const int nitems = ntx * nty * ntz * a.nsamp;
    for (int it = blockIdx.x; it < nitems; it += gridDim.x) {
        int r = it;
        const int tx = r % ntx;
        r /= ntx;
        const int ty = r % nty;
        r /= nty;
        const int tz = r % ntz;
        const int smp = r / ntz;
        const int x0 = tx * 16, y0 = ty * TR, z0 = tz * WG_ZC, ze = min(z0 + WG_ZC, g.nz);
        const size_t sbase = (size_t)smp * g.ncell;

        // Per item, each lane's staging chunks sit at fixed offsets within a
        // plane (global) and within a buffer (LDS); a plane adds its offset.
        // Chunk v of an act plane: channel group v % NCG of cell (v / NCG) % 18
        // (x0 - 1 + cell) in row v / (18 NCG) (y0 - 1 + row, which wraps more than
        // once where ny < TR + 1); chunk t of a dz plane, RD of them per lane: group
        // t % NCGZ, cell (t / NCGZ) % 16, row t / (16 NCGZ) (rows past ny contribute
        // zero). Act plane p and dz plane p + 1 go to slot (p - z0 + 1) mod 3.
        const size_t plane_a = (size_t)g.ny * g.nx * CIN, plane_d = (size_t)g.ny * g.nx * COUTS;
        const u16 *act_s = a.act + sbase * CIN, *dz_s = a.dz + sbase * COUTS;
        uint32_t goff_a[RA]; // in 16-byte chunks
        int loff_a[RA];
#pragma unroll
        for (int k = 0; k < RA; ++k) {
            const int v = min(tid + 256 * k, T_ACT - 1);
            const int cg = v % NCG, cell = (v / NCG) % 18, row = v / (18 * NCG);
            const int x = wrapc(x0 + cell - 1, g.nx);
            int y = y0 + row - 1;
            if (y < 0) y += g.ny;
            while (y >= g.ny) y -= g.ny;
            goff_a[k] = ((uint32_t)y * g.nx + x) * NCG + cg;
            loff_a[k] = row * AROW + wg_pos(cell, 8 * cg);
        }
        // rows past ny load a valid chunk of the plane and store zero
        bool dz_in[RD];
        uint32_t goff_d[RD];
        int loff_d[RD];
#pragma unroll
        for (int r = 0; r < RD; ++r) {
            const int t = tid + 256 * r;
            const int dcg = t % NCGZ, dcell = (t / NCGZ) % 16, drow = t / (16 * NCGZ);
            dz_in[r] = y0 + drow < g.ny;
            goff_d[r] = ((uint32_t)(dz_in[r] ? y0 + drow : 0) * g.nx + x0 + dcell) * NCGZ + dcg;
            loff_d[r] = drow * DROW + wg_pos(dcell, 8 * dcg);
        }

        // Act plane q and dz plane q + 1 travel together; qa and qd hold the pair
        // for one step between its loads and its stores. Every step issues the same
        // loads and stores (plane indices clamped to the chunk; dz planes outside it are
        // stored as zeros), and nothing touches the loaded values before the stores,
        // so that the loads stay in flight.
        u32x4 qa[RA], qd[RD];
        auto load = [&](int q) __attribute__((always_inline)) {
            const u32x4 *pa = reinterpret_cast<const u32x4 *>(act_s + (size_t)wrapc(min(q, ze), g.nz) * plane_a);
#pragma unroll
            for (int k = 0; k < RA; ++k) qa[k] = pa[goff_a[k]];
            const u32x4 *pd = reinterpret_cast<const u32x4 *>(dz_s + (size_t)min(q + 1, ze - 1) * plane_d);
#pragma unroll
            for (int r = 0; r < RD; ++r) qd[r] = pd[goff_d[r]];
        };
        auto store = [&](int q, int slot) __attribute__((always_inline)) {
#pragma unroll
            for (int k = 0; k < RA; ++k) *reinterpret_cast<u32x4 *>(act_l + slot * APL + loff_a[k]) = qa[k];
#pragma unroll
            for (int r = 0; r < RD; ++r) { // chunk r of this lane: channel group tid % NCGZ, as every r
                const u32x4 w = dz_in[r] && q + 1 < ze ? qd[r] : u32x4{0u, 0u, 0u, 0u};
#pragma unroll
                for (int c = 0; c < 8; ++c) bs[c] += bf2f((u16)((c & 1) ? (w[c >> 1] >> 16) : (w[c >> 1] & 0xffffu)));
                *reinterpret_cast<u32x4 *>(dz_l + slot * DPL + loff_d[r]) = w;
            }
        };
        // dz fragments (K chunk c) of plane p in f[(p - z0 + 1) mod 3]
        bf16x8 f[3][NKC];
#pragma unroll
        for (int c = 0; c < NKC; ++c) f[0][c] = f[1][c] = f[2][c] = bf16x8{};

        // B fragment k = e NKC + c of a plane: offset pair e (y, x), K chunk c, from the
        // act plane in `slot`, into a window of NB fragments.
        constexpr int NB = 6, NK = 9 * NKC;
        static_assert(NKC == 4 && NK % NB == 0, "the window's positions repeat every plane");
        bf16x8 b[NB];
        auto read_b = [&](int slot, int k) __attribute__((always_inline)) {
            const int e = k / NKC, c = k % NKC, dyo = e / 3 - 1, dxo = e % 3 - 1;
            b[k % NB] = frag_tr(act_l + slot * APL + (2 * c + (quad >> 1) + dyo + 1) * AROW, 8 * (quad & 1) + dxo + 1, 16 * nw, col);
        };
        // Step J of three (slots, fragment sets): act plane p, in slot J, meets dz planes
        // p + 1 (z offset -1), p (0) and p - 1 (+1); the fragments of planes outside
        // [z0, ze) are zero (one code path: the planes around a chunk cost MFMAs that
        // add exact zeros). A B fragment is read five fragments, 15 MFMAs, ahead of its
        // own, the next plane's first ones in this step; plane p + 1's dz fragments are
        // read here and meet the first offset pair last. Half way every wavefront has
        // left plane p - 1: the planes p + 2 take its slot.
        auto step = [&](auto j, int p) __attribute__((always_inline)) {
            constexpr int J = decltype(j)::value, J1 = (J + 1) % 3, J2 = (J + 2) % 3;
#pragma unroll
            for (int c = 0; c < NKC; ++c) f[J1][c] = frag_tr(dz_l + J * DPL + (2 * c + (quad >> 1)) * DROW, 8 * (quad & 1), 16 * mw, col);
            read_b(J, 5);
#pragma unroll
            for (int c = 0; c < NKC; ++c) {
                acc[9] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f[J][c], b[c], acc[9], 0, 0, 0);
                acc[18] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f[J2][c], b[c], acc[18], 0, 0, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int c = 0; c < NKC; ++c) acc[0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f[J1][c], b[c], acc[0], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int k = NKC; k < NK; ++k) {
                const int e = k / NKC, c = k % NKC;
#pragma unroll
                for (int n = k == NKC ? 6 : k + 5; n <= k + 5; ++n)
                    if (n < NK) read_b(J, n);
                    else read_b(J1, n - NK);
                acc[e] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f[J1][c], b[k % NB], acc[e], 0, 0, 0);
                acc[9 + e] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f[J][c], b[k % NB], acc[9 + e], 0, 0, 0);
                acc[18 + e] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f[J2][c], b[k % NB], acc[18 + e], 0, 0, 0);
                if (k == NK / 2) {
                    wg_lds_barrier();
                    store(p + 2, J2);
                    load(p + 3);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        };

        load(z0 - 1);
        store(z0 - 1, 0);
        load(z0);
        store(z0, 1);
        load(z0 + 1);
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 5; ++k) read_b(0, k);
        for (int p = z0 - 1; p <= ze; p += 3) { // (a chunk's planes and two, rounded up to three)
            step(IntC<0>{}, p);
            step(IntC<1>{}, p + 1);
            step(IntC<2>{}, p + 2);
        }
        __syncthreads(); // the slots are free
    }

    // Bias partials: dz staging lane t summed channels 8 (t % NCGZ) + c (of
    // every chunk it stages); fold the lanes of each channel in lane order.
#pragma unroll
    for (int c = 0; c < 8; ++c) bsum_l[tid][c] = bs[c];
    __syncthreads();
    if (tid < COUTS) {
        float t = 0.f;
        for (int l = tid / 8; l < 256; l += NCGZ) t += bsum_l[l][tid % 8];
        a.bpart[(size_t)blockIdx.x * 32 + tid] = t;
    }
    // acc[d][j]: co = 16 mw + 4 quad + j, ci = 16 nw + col
    constexpr int PCO = 16 * MT, PCI = 16 * NT;
    float *part = a.part + (size_t)blockIdx.x * 27 * PCO * PCI;
#pragma unroll
    for (int d = 0; d < 27; ++d)
#pragma unroll
        for (int j = 0; j < 4; ++j) part[((size_t)d * PCO + 16 * mw + 4 * quad + j) * PCI + 16 * nw + col] = acc[d][j];
}

// Weight gradients of the first layer (8 -> 32 stored channels) and of the last
// (32 -> 8, two of them real). One side has few channels, and as a product per
// offset (wgrad_kernel) they fill little of an MFMA tile. Here the rows of the
// product are the pairs (offset, channel) of the narrow side, shifted, and the
// columns the 32 channels of the wide side, unshifted:
//   last layer:  rows 2 d + co, dz[p - d][co] against act[p][ci];
//   first layer: rows 4 d + s,  x[c + d][s] against dz[c][co], s the high and low
//                parts of u and v; the (F, k) channels are constant over a
//                sample, so their gradient is the same for every offset: two
//                rows of constants, and a row of ones gives the bias gradient.
// 4 (last) or 7 (first) row tiles by two column tiles per K = 32 cells: 8 and 14
// MFMAs where the offset-by-offset kernel takes 54, and the wide tensor, which is
// not shifted, is read once and without a halo.
//
// Every wavefront works alone (no barriers until its sums are folded): it owns
// patches of 16 x-cells by 4 rows through a chunk of planes, stages the wide
// tensor's plane channels-last in LDS (read back as fragments of 8 cells per
// channel, frag_tr), and the narrow one planar, in three copies shifted by one
// cell, so that a row's fragment is one aligned 16-byte read. Loads run a plane
// ahead. What bounds it: the read of the wide tensor (0.54 GB at 4 x 128^3, with
// the 0.13 GB of the narrow one 0.13 ms at the rate of a large copy). 4 x 128^3:
// last layer 430 -> 157 us, first layer 268 -> 140 (its narrow side is read at
// four of its eight channels, with 45 KB of LDS per workgroup three per CU).
constexpr int WS_RT = 4;      // rows of a patch
constexpr int WS_WAVES = 4;   // wavefronts of a workgroup
template <bool FIRST> struct WsGeom {
    static constexpr int NS = FIRST ? 4 : 2;                 // shifted channels
    static constexpr int CONST0 = 27 * NS;                   // first layer: rows of ones, F, k; last: bias rows
    static constexpr int MT = (CONST0 + (FIRST ? 3 : 0) + 15) / 16;
    static constexpr int ROWS = 16 * MT;                     // rows of a partial (x 32 columns)
    static constexpr int U16 = WS_RT * 16 * 32;              // wide plane (16-bit units)
    static constexpr int SROW = NS * 3 * 16;                 // narrow plane: [row][channel][copy][cell]
    static constexpr int SLOT = (WS_RT + 2) * SROW + (FIRST ? 48 : 0); // a plane slot, with the constant rows
    static constexpr int WAVE16 = U16 + 3 * SLOT;
};
template <bool FIRST>
__global__ __launch_bounds__(64 * WS_WAVES) void wgrad_shift_kernel(WgradArgs a)
{
    typedef WsGeom<FIRST> G;
    constexpr int NS = G::NS, MT = G::MT;
    __shared__ __align__(16) u16 lds[WS_WAVES * G::WAVE16];
    static_assert(sizeof(lds) >= 2 * MT * 2 * 256 * 4, "two wavefronts' sums fit");
    const Geo g = a.geo;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int col = lane & 15, quad = lane >> 4;
    u16 *ul = lds + wave * G::WAVE16, *sl = ul + G::U16;
    const u16 *wide = FIRST ? a.dz : a.act, *narrow = FIRST ? a.act : a.dz;

    f32x4 acc[MT][2];
#pragma unroll
    for (int t = 0; t < MT; ++t)
#pragma unroll
        for (int n = 0; n < 2; ++n) acc[t][n] = f32x4{0.f, 0.f, 0.f, 0.f};
    float bs[2] = {0.f, 0.f}; // last layer: the lane's sums of dz

    // Row 16 t + col of the product: its place in a narrow slot (without the
    // cell group and the patch row) and its plane offset plus one.
    int srow[MT], soz[MT], sky[MT];
#pragma unroll
    for (int t = 0; t < MT; ++t) {
        const int r = 16 * t + col;
        const int d = min(r / NS, 26), ch = r % NS;
        const int dz = d / 9, dy = d / 3 % 3, dx = d % 3;
        const int ox = FIRST ? dx - 1 : 1 - dx, oy = FIRST ? dy - 1 : 1 - dy, oz = FIRST ? dz - 1 : 1 - dz;
        const bool con = FIRST && r >= G::CONST0;
        srow[t] = con ? (WS_RT + 2) * G::SROW + min(r - G::CONST0, 2) * 16 : ((oy + 1) * NS + ch) * 48 + (ox + 1) * 16;
        soz[t] = oz + 1;
        sky[t] = con ? 0 : G::SROW; // the step per patch row
    }
    const int ntx = g.nx / 16, nty = (g.ny + WS_RT - 1) / WS_RT, ntz = (g.nz + a.zc - 1) / a.zc;
    const int nitems = ntx * nty * ntz * a.nsamp;
    for (int it = blockIdx.x * WS_WAVES + wave; it < nitems; it += gridDim.x * WS_WAVES) {
        int r = it;
        const int tx = r % ntx;
        r /= ntx;
        const int ty = r % nty;
        r /= nty;
        const int tz = r % ntz, smp = r / ntz;
        const int x0 = 16 * tx, y0 = WS_RT * ty, z0 = tz * a.zc, ze = min(z0 + a.zc, g.nz);
        const size_t sbase = (size_t)smp * g.ncell, plane = (size_t)g.nx * g.ny;

        // Wide: load k is patch row k, lane = cell 4 (lane / 4) .. of 16-byte
        // chunks (rows past ny read a valid row and count as zero).
        size_t uoff[WS_RT];
#pragma unroll
        for (int k = 0; k < WS_RT; ++k) uoff[k] = ((size_t)min(y0 + k, g.ny - 1) * g.nx + x0) * 32 + lane * 8;
        const int upos = wg_pos(lane >> 2, 8 * (lane & 3));
        // Narrow: load k is cell v = lane + 64 k of the 18 x 6 cells around the patch.
        size_t soff[2];
        int srx[2], sry[2];
        bool inner[2];
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const int v = min(lane + 64 * k, 18 * (WS_RT + 2) - 1);
            srx[k] = v % 18;
            sry[k] = v / 18;
            int y = y0 + sry[k] - 1;
            y = y < 0 ? y + g.ny : y;
            while (y >= g.ny) y -= g.ny;
            soff[k] = ((size_t)y * g.nx + wrapc(x0 + srx[k] - 1, g.nx)) * 8;
            inner[k] = lane + 64 * k < 18 * (WS_RT + 2) && srx[k] >= 1 && srx[k] <= 16 && sry[k] >= 1 && sry[k] <= WS_RT &&
                       y0 + sry[k] - 1 < g.ny;
        }
        uint4 qu[WS_RT], qs[2];
        auto load_u = [&](int z) __attribute__((always_inline)) {
            const u16 *p = wide + (sbase + (size_t)z * plane) * 32;
#pragma unroll
            for (int k = 0; k < WS_RT; ++k) qu[k] = *reinterpret_cast<const uint4 *>(p + uoff[k]);
        };
        auto load_s = [&](int z) __attribute__((always_inline)) {
            const u16 *p = narrow + (sbase + (size_t)wrapc(z, g.nz) * plane) * 8;
#pragma unroll
            for (int k = 0; k < 2; ++k) qs[k] = *reinterpret_cast<const uint4 *>(p + soff[k]);
        };
        auto store_u = [&]() __attribute__((always_inline)) {
#pragma unroll
            for (int k = 0; k < WS_RT; ++k)
                *reinterpret_cast<uint4 *>(ul + k * 512 + upos) = y0 + k < g.ny ? qu[k] : uint4{0u, 0u, 0u, 0u};
        };
        // Narrow plane z into slot `slot`; copy c holds cell x0 + i + c - 1 at i.
        auto store_s = [&](int slot, bool own) __attribute__((always_inline)) {
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const u16 ch[4] = {(u16)(qs[k].x & 0xffffu), (u16)(qs[k].x >> 16), (u16)(qs[k].z & 0xffffu), (u16)(qs[k].z >> 16)};
                u16 *dst = sl + slot * G::SLOT + sry[k] * G::SROW;
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    const int i = srx[k] - c;
                    if (i >= 0 && i < 16 && lane + 64 * k < 18 * (WS_RT + 2))
#pragma unroll
                        for (int s = 0; s < NS; ++s) dst[(s * 3 + c) * 16 + i] = ch[s];
                }
                if (!FIRST && own && inner[k]) {
                    bs[0] += bf2f(ch[0]);
                    bs[1] += bf2f(ch[1]);
                }
            }
        };
        // slots: plane z in ((z - z0) + 3) mod 3
        load_s(z0 - 1);
        if constexpr (FIRST) {
            // constant rows of every slot: ones, F, k (channels 2 and 3 of any cell of the sample)
            const uint32_t fk = __shfl(qs[0].y, 0, 64);
            if (lane < 48) {
                const u16 v = lane < 16 ? (u16)0x3F80 : lane < 32 ? (u16)(fk & 0xffffu) : (u16)(fk >> 16);
#pragma unroll
                for (int p = 0; p < 3; ++p) sl[p * G::SLOT + (WS_RT + 2) * G::SROW + lane] = v;
            }
        }
        store_s(2, false);
        load_s(z0);
        store_s(0, true);
        load_u(z0);
        load_s(z0 + 1);
        int ph = 0; // (z - z0) mod 3
        for (int z = z0; z < ze; ++z) {
            store_u();
            store_s(ph == 2 ? 0 : ph + 1, z + 1 < ze);
            __builtin_amdgcn_wave_barrier(); // the fragment reads below follow the stores (LDS keeps a wavefront's order)
            load_u(min(z + 1, ze - 1));
            load_s(min(z + 2, ze));
#pragma unroll
            for (int c = 0; c < WS_RT / 2; ++c) {
                const int prow = 2 * c + (quad >> 1), cell0 = 8 * (quad & 1);
                bf16x8 b[2];
#pragma unroll
                for (int n = 0; n < 2; ++n) b[n] = frag_tr(ul + prow * 512, cell0, 16 * n, col);
#pragma unroll
                for (int t = 0; t < MT; ++t) {
                    // slot of plane z + soz - 1
                    int q = ph + soz[t] + 2;
                    q = q >= 3 ? q - 3 : q;
                    q = q >= 3 ? q - 3 : q;
                    const bf16x8 av = load8(sl + q * G::SLOT + srow[t] + prow * sky[t] + cell0);
#pragma unroll
                    for (int n = 0; n < 2; ++n) acc[t][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, b[n], acc[t][n], 0, 0, 0);
                }
            }
            ph = ph == 2 ? 0 : ph + 1;
        }
    }

    // Fold the wavefronts' sums: 2 and 3 into 0 and 1, then 1 into 0; wavefront 0
    // writes the workgroup's partial. acc[t][n][j]: row 16 t + 4 quad + j, column
    // 16 n + col.
    float *red = reinterpret_cast<float *>(lds);
#pragma unroll
    for (int h = 2; h >= 1; h /= 2) {
        __syncthreads();
        if (wave >= h && wave < 2 * h)
#pragma unroll
            for (int t = 0; t < MT; ++t)
#pragma unroll
                for (int n = 0; n < 2; ++n)
                    *reinterpret_cast<f32x4 *>(red + (((wave - h) * MT + t) * 2 + n) * 256 + lane * 4) = acc[t][n];
        __syncthreads();
        if (wave < h)
#pragma unroll
            for (int t = 0; t < MT; ++t)
#pragma unroll
                for (int n = 0; n < 2; ++n) acc[t][n] += *reinterpret_cast<const f32x4 *>(red + ((wave * MT + t) * 2 + n) * 256 + lane * 4);
    }
    float *part = a.part + (size_t)blockIdx.x * G::ROWS * 32;
    if constexpr (!FIRST) {
        // bias sums into the spare rows 54 and 55, column 0: lanes in order, then wavefronts
        __syncthreads();
        red[2 * threadIdx.x] = bs[0];
        red[2 * threadIdx.x + 1] = bs[1];
        __syncthreads();
    }
    if (wave == 0) {
#pragma unroll
        for (int t = 0; t < MT; ++t)
#pragma unroll
            for (int n = 0; n < 2; ++n)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int r = 16 * t + 4 * quad + j;
                    if (FIRST || r < G::CONST0) part[r * 32 + 16 * n + col] = acc[t][n][j];
                }
        if (!FIRST && lane < 2) {
            float s = 0.f;
            for (int i = 0; i < 64 * WS_WAVES; ++i) s += red[2 * i + lane];
            part[(G::CONST0 + lane) * 32] = s;
        }
    }
}

// Gradients of the first or last layer from wgrad_shift_kernel's partials: one
// workgroup per output row of 32 columns, 8 slices of the partials summed in
// FP64 and folded in a fixed order.
// FIRST: blocks 0 .. 53: (offset, u or v), the high and the low part's rows;
// 54, 55: F and k (one row each, the same for every offset); 56: the bias.
// Last: blocks 0 .. 53: row 2 d + co; 54, 55: the bias of channel 0, 1.
template <bool FIRST>
__global__ __launch_bounds__(256) void wgrad_shift_reduce(const float *__restrict__ part, int nblk, float *__restrict__ gW,
                                                          float *__restrict__ gb)
{
    typedef WsGeom<FIRST> G;
    __shared__ double red[8][32];
    const int c = threadIdx.x & 31, j = threadIdx.x >> 5, o = blockIdx.x;
    const int d = o / 2, ch = o % 2;
    const int row = !FIRST ? (o < 54 ? o : G::CONST0 + ch) : o < 54 ? 4 * d + ch : o < 56 ? G::CONST0 + 1 + ch : G::CONST0;
    double s = 0.0;
    const float *p = part + (size_t)row * 32 + c;
    // unrolled so that eight loads are in flight; the adds keep their order
#pragma unroll 8
    for (int b = j; b < nblk; b += 8) s += p[(size_t)b * (G::ROWS * 32)];
    if (FIRST && o < 54)
#pragma unroll 8
        for (int b = j; b < nblk; b += 8) s += p[(size_t)b * (G::ROWS * 32) + 2 * 32];
    red[j][c] = s;
    __syncthreads();
    if (j != 0) return;
    double t = 0.0;
    for (int i = 0; i < 8; ++i) t += red[i][c];
    const float v = (float)t;
    if constexpr (FIRST) {
        // W[co = c][ci][d], 4 input channels
        if (o < 54) gW[(c * 4 + ch) * 27 + d] = v;
        else if (o < 56)
            for (int e = 0; e < 27; ++e) gW[(c * 4 + 2 + ch) * 27 + e] = v;
        else gb[c] = v;
    } else {
        // W[co = ch][ci = c][d]
        if (o < 54) gW[(ch * 32 + c) * 27 + d] = v;
        else if (c == 0) gb[ch] = v;
    }
}

// grad[W(co, ci, d)] of a 32 -> 32 layer = sum over workgroups of the partials.
// A workgroup handles 64 outputs (input channel fastest, so the loads of a wave
// are contiguous) with 4 slices each: slice j sums the workgroups b = j, j + 4,
// ... in order, and the 4 slice sums are added in a fixed order: the result does
// not depend on scheduling.
__global__ __launch_bounds__(256) void wgrad_reduce(const float *__restrict__ part, int nblk, float *__restrict__ gW)
{
    __shared__ double red[4][64];
    const int o = threadIdx.x & 63, j = threadIdx.x >> 6;
    const int e = blockIdx.x * 64 + o; // (d, co, ci)
    double s = 0.0;
    // unrolled so that eight loads are in flight; the adds keep their order
#pragma unroll 8
    for (int b = j; b < nblk; b += 4) s += part[(size_t)b * (27 * 32 * 32) + e];
    red[j][o] = s;
    __syncthreads();
    const int ci = e % 32, co = e / 32 % 32, d = e / 1024;
    if (j == 0) gW[(co * 32 + ci) * 27 + d] = (float)((red[0][o] + red[1][o]) + (red[2][o] + red[3][o]));
}

// Bias gradient: fixed-order fold of the per-workgroup channel sums; 32
// groups of lanes each sum every 32nd workgroup in order, then lane c adds
// the 32 group sums of channel c in order.
__global__ __launch_bounds__(1024) void colsum_reduce(const float *__restrict__ part, int nblk, float *__restrict__ gb)
{
    __shared__ double red[32][32];
    const int c = threadIdx.x & 31, g = threadIdx.x >> 5;
    double s = 0.0;
    for (int b = g; b < nblk; b += 32) s += part[(size_t)b * 32 + c];
    red[g][c] = s;
    __syncthreads();
    if (g == 0) {
        double t = 0.0;
        for (int i = 0; i < 32; ++i) t += red[i][c];
        gb[c] = (float)t;
    }
}

// ------------------------------------------------------------------ input, loss, optimiser
template <typename IO>
__global__ __launch_bounds__(256) void pack_input(const IO *__restrict__ u, const IO *__restrict__ v,
                                                  FkArgs fk, int nsamp, int ncell, u16 *__restrict__ x)
{
    const size_t rows = (size_t)nsamp * ncell;
    for (size_t r = (size_t)blockIdx.x * blockDim.x + threadIdx.x; r < rows; r += (size_t)gridDim.x * blockDim.x) {
        const int s = (int)(r / ncell);
        // u and v as BF16 pairs hi + lo (about 16 significant bits); the first
        // layer applies the same weight to both parts.
        const float uf = (float)u[r], vf = (float)v[r];
        const u16 uh = f2bf(uf), vh = f2bf(vf);
        const u16 ul = f2bf(uf - bf2f(uh)), vl = f2bf(vf - bf2f(vh));
        uint4 q;
        q.x = (uint32_t)uh | ((uint32_t)vh << 16);
        q.y = (uint32_t)f2bf((fk.f[s] - F_CENTER) / F_SCALE) | ((uint32_t)f2bf((fk.k[s] - K_CENTER) / K_SCALE) << 16);
        q.z = (uint32_t)ul | ((uint32_t)vl << 16);
        q.w = 0u;
        *reinterpret_cast<uint4 *>(x + r * 8) = q;
    }
}

// Residuals of the prediction, their squared sum per workgroup, and the loss
// gradient dL/dpred = 2 (pred - target) / n_terms (channels 0, 1 of 8).
__global__ __launch_bounds__(256) void loss_grad(const float *__restrict__ pu, const float *__restrict__ pv,
                                                 const float *__restrict__ tu, const float *__restrict__ tv,
                                                 size_t rows, float scale, u16 *__restrict__ dz4,
                                                 double *__restrict__ part)
{
    __shared__ double red[256];
    double acc = 0.0;
    for (size_t r = (size_t)blockIdx.x * blockDim.x + threadIdx.x; r < rows; r += (size_t)gridDim.x * blockDim.x) {
        const float ru = pu[r] - tu[r], rv = pv[r] - tv[r];
        acc += (double)ru * ru + (double)rv * rv;
        uint4 q;
        q.x = (uint32_t)f2bf(scale * ru) | ((uint32_t)f2bf(scale * rv) << 16);
        q.y = q.z = q.w = 0u;
        *reinterpret_cast<uint4 *>(dz4 + r * 8) = q;
    }
    red[threadIdx.x] = acc;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}

__global__ __launch_bounds__(256) void adam_kernel(float *__restrict__ p, const float *__restrict__ gr,
                                                   float *__restrict__ m, float *__restrict__ v, int n, float lr,
                                                   float b1, float b2, float eps, float c1, float c2)
{
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
        const float g = gr[i];
        const float mi = b1 * m[i] + (1.f - b1) * g;
        const float vi = b2 * v[i] + (1.f - b2) * g * g;
        m[i] = mi;
        v[i] = vi;
        p[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
    }
}

// Packs layer weights (FP32, W[co][ci][d]) into the B-fragment order of the
// convolution kernel: chunk c, N-tile t, lane, 8 consecutive k = 32 c + 8
// (lane / 16) + j with k = d * cins + ci. DGRAD packs the mirrored, transposed
// weights W'[ci][co][d] = W[co][ci][26 - d] (input channels = co).
// lo_pairs: input channels cin .. cin + lo_pairs - 1 carry the low parts of
// channels 0 .. lo_pairs - 1 and take their weights.
__global__ __launch_bounds__(256) void repack(const float *__restrict__ W, int cout, int cin, int cins, int nch,
                                              int dgrad, int lo_pairs, u16 *__restrict__ out)
{
    constexpr int NT = 2;
    const int total = nch * NT * 64 * 8;
    for (int e = blockIdx.x * blockDim.x + threadIdx.x; e < total; e += gridDim.x * blockDim.x) {
        const int j = e % 8, lane = (e / 8) % 64, t = (e / 512) % NT, c = e / (512 * NT);
        const int k = 32 * c + 8 * (lane / 16) + j;
        // row m of tile t is output channel 8 (m / 4) + 4 t + m % 4, so that a lane's
        // accumulators of both tiles are 8 consecutive channels
        const int m = lane % 16;
        const int d = k / cins, kc = k % cins, n = 8 * (m / 4) + 4 * t + m % 4;
        float w = 0.f;
        if (d < 27) {
            if (!dgrad) {
                const int src = kc < cin ? kc : (kc - cin < lo_pairs ? kc - cin : -1);
                if (src >= 0 && n < cout) w = W[((size_t)n * cin + src) * 27 + d];
            } else {
                // input channel kc = co of the layer, output channel n = ci of the layer
                if (kc < cout && n < cin) w = W[((size_t)kc * cin + n) * 27 + (26 - d)];
            }
        }
        out[e] = f2bf(w);
    }
}

// Weights of the output layer for conv_out_kernel: fragment 2 dz + t, row m of
// tile t is offset (16 t + m) / 2 of the nine (dy, dx) and output channel m % 2
// (rows past 17 are zero), 8 consecutive input channels per lane.
__global__ __launch_bounds__(256) void repack_out(const float *__restrict__ W, u16 *__restrict__ out)
{
    const int e = blockIdx.x * 256 + threadIdx.x; // 6 x 64 x 8
    const int j = e % 8, lane = e / 8 % 64, t = e / 512 % 2, dz = e / 1024;
    if (dz >= 3) return;
    const int r = 16 * t + lane % 16, ci = 8 * (lane / 16) + j;
    out[e] = r < 18 ? f2bf(W[((size_t)(r % 2) * 32 + ci) * 27 + 9 * dz + r / 2]) : (u16)0;
}

// ------------------------------------------------------------------ launchers
static int grid_cap(size_t work, int per_block, int cap)
{
    size_t b = (work + per_block - 1) / per_block;
    if (b < 1) b = 1;
    if (b > (size_t)cap) b = cap;
    return (int)b;
}

// The chunk of planes with the fewest plane times for `cols` columns of work on
// `slots` places: rounds of chunks times a chunk's planes and the two more it
// reads.
static int balanced_zc(int nz, size_t cols, size_t slots)
{
    int best = 1;
    size_t cost = ~(size_t)0;
    for (int n = 1; n <= nz && n <= 64; ++n) {
        const int zc = (nz + n - 1) / n;
        const size_t items = cols * ((nz + zc - 1) / zc), c = (items + slots - 1) / slots * (zc + 2);
        if (c < cost) {
            cost = c;
            best = zc;
        }
    }
    return best;
}

// Planes per workgroup of conv8_kernel and conv32p_kernel, a multiple of `unit` (the
// phases their steps rotate over); the last chunk ends with the grid and may repeat
// planes of the one before, with the same results. The chunk is the one with the
// fewest plane times on `slots` places, where the weights' load and the first planes
// count as two.
static int chunk_planes(int nz, size_t cols, size_t slots, int unit)
{
    int best = unit;
    size_t cost = ~(size_t)0;
    for (int n = 1; n <= nz / unit && n <= 1024; ++n) {
        const int zc = std::min((nz + unit * n - 1) / (unit * n), nz / unit) * unit;
        const size_t c = (cols * ((nz + zc - 1) / zc) + slots - 1) / slots * (zc + 2);
        if (c < cost) {
            cost = c;
            best = zc;
        }
    }
    return best;
}

hipError_t launch_conv(int cin, int mode, int io_f64, const ConvArgs &a, int cus, hipStream_t st)
{
    if (a.geo.nx % PX != 0 || a.geo.nz < 4) return hipErrorInvalidValue;
    if (mode != MODE_OUT && (cin == 8 || cin == 32)) {
        ConvArgs b = a;
        const int waves = cin == 8 ? C8_WAVES : C32_WAVES, py = waves * (cin == 8 ? C8_RW : C32_RW);
        const size_t cols = (size_t)(a.geo.nx / PX) * ((a.geo.ny + py - 1) / py) * a.nsamp;
        // workgroups at once: three of conv8_kernel a CU (registers), one of
        // conv32p_kernel (registers and LDS)
        b.zc = cin == 8 ? chunk_planes(a.geo.nz, cols, 3 * (size_t)cus, 3) : chunk_planes(a.geo.nz, cols, cus, 4);
        const size_t nb = cols * ((a.geo.nz + b.zc - 1) / b.zc);
        if (nb == 0 || nb > 0x7fffffffu) return hipErrorInvalidConfiguration;
        auto go = [&](auto m) {
            constexpr int M = decltype(m)::value;
            if (cin == 8) hipLaunchKernelGGL(conv8_kernel<M>, dim3((unsigned)nb), dim3(64 * waves), 0, st, b);
            else hipLaunchKernelGGL(conv32p_kernel<M>, dim3((unsigned)nb), dim3(64 * waves), 0, st, b);
            return hipGetLastError();
        };
        return mode == MODE_HIDDEN ? go(IntC<MODE_HIDDEN>{}) : mode == MODE_ACT ? go(IntC<MODE_ACT>{}) : go(IntC<MODE_DGRAD>{});
    }
    if (cin == 32 && mode == MODE_OUT) {
        ConvArgs b = a;
        const int ng = a.geo.nx / 16, tg = ng <= OUT_NG ? ng : OUT_NG - 2;
        const size_t cols = (size_t)((ng + tg - 1) / tg) * ((a.geo.ny + OUT_TY - 1) / OUT_TY) * a.nsamp;
        b.zc = balanced_zc(a.geo.nz, cols, cus); // one workgroup per CU
        const size_t nb = cols * ((a.geo.nz + b.zc - 1) / b.zc);
        if (nb == 0 || nb > 0x7fffffffu) return hipErrorInvalidConfiguration;
        auto go = [&](auto full) {
            if (io_f64) hipLaunchKernelGGL((conv_out_kernel<double, decltype(full)::value>), dim3((unsigned)nb), dim3(512), 0, st, b);
            else hipLaunchKernelGGL((conv_out_kernel<float, decltype(full)::value>), dim3((unsigned)nb), dim3(512), 0, st, b);
            return hipGetLastError();
        };
        return ng >= OUT_NG ? go(BoolC<true>{}) : go(BoolC<false>{});
    }
    return hipErrorInvalidValue;
}

int wgrad_blocks() { return 512; }

hipError_t launch_wgrad_edge(bool first, const WgradArgs &a, float *gW, float *gb, int cus, hipStream_t st)
{
    // resident at once: 3 workgroups per CU (LDS), or 4; the partials have room for 1024
    const size_t slots = std::min<size_t>((first ? 3 : 4) * (size_t)cus, 1024);
    const size_t cols = (size_t)(a.geo.nx / 16) * ((a.geo.ny + WS_RT - 1) / WS_RT) * a.nsamp;
    WgradArgs b = a;
    b.zc = balanced_zc(a.geo.nz, cols, slots * WS_WAVES);
    const size_t items = cols * ((a.geo.nz + b.zc - 1) / b.zc);
    if (items == 0 || items > 0x7fffffffu) return hipErrorInvalidConfiguration;
    const int grid = (int)std::min<size_t>(slots, (items + WS_WAVES - 1) / WS_WAVES);
    if (first) {
        hipLaunchKernelGGL(wgrad_shift_kernel<true>, dim3(grid), dim3(64 * WS_WAVES), 0, st, b);
        hipLaunchKernelGGL(wgrad_shift_reduce<true>, dim3(57), dim3(256), 0, st, b.part, grid, gW, gb);
    } else {
        hipLaunchKernelGGL(wgrad_shift_kernel<false>, dim3(grid), dim3(64 * WS_WAVES), 0, st, b);
        hipLaunchKernelGGL(wgrad_shift_reduce<false>, dim3(56), dim3(256), 0, st, b.part, grid, gW, gb);
    }
    return hipGetLastError();
}

hipError_t launch_wgrad(const WgradArgs &a, hipStream_t st)
{
    hipLaunchKernelGGL(wgrad_kernel, dim3(wgrad_blocks()), dim3(256), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_wgrad_reduce(const float *part, float *gW, hipStream_t st)
{
    hipLaunchKernelGGL(wgrad_reduce, dim3(32 * 32 * 27 / 64), dim3(256), 0, st, part, wgrad_blocks(), gW);
    return hipGetLastError();
}

hipError_t launch_bias_reduce(const float *bpart, float *gb, hipStream_t st)
{
    hipLaunchKernelGGL(colsum_reduce, dim3(1), dim3(1024), 0, st, bpart, wgrad_blocks(), gb);
    return hipGetLastError();
}

hipError_t launch_pack_input(int io_f64, const void *u, const void *v, const FkArgs &fk, int nsamp, int ncell,
                             uint16_t *x, hipStream_t st)
{
    const int grid = grid_cap((size_t)nsamp * ncell, 256, 65536);
    if (io_f64)
        hipLaunchKernelGGL(pack_input<double>, dim3(grid), dim3(256), 0, st, (const double *)u, (const double *)v, fk,
                           nsamp, ncell, x);
    else
        hipLaunchKernelGGL(pack_input<float>, dim3(grid), dim3(256), 0, st, (const float *)u, (const float *)v, fk,
                           nsamp, ncell, x);
    return hipGetLastError();
}

int loss_blocks() { return 1024; }

hipError_t launch_loss_grad(const float *pu, const float *pv, const float *tu, const float *tv, size_t rows,
                            float scale, uint16_t *dz4, double *part, hipStream_t st)
{
    hipLaunchKernelGGL(loss_grad, dim3(loss_blocks()), dim3(256), 0, st, pu, pv, tu, tv, rows, scale, dz4, part);
    return hipGetLastError();
}

hipError_t launch_adam(float *p, const float *g, float *m, float *v, int n, float lr, float b1, float b2, float eps,
                       float c1, float c2, hipStream_t st)
{
    hipLaunchKernelGGL(adam_kernel, dim3(grid_cap(n, 256, 1024)), dim3(256), 0, st, p, g, m, v, n, lr, b1, b2, eps,
                       c1, c2);
    return hipGetLastError();
}

hipError_t launch_repack_out(const float *W, uint16_t *out, hipStream_t st)
{
    hipLaunchKernelGGL(repack_out, dim3(12), dim3(256), 0, st, W, out);
    return hipGetLastError();
}

hipError_t launch_repack(const float *W, int cout, int cin, int cins, int nch, int dgrad, int lo_pairs, uint16_t *out,
                         hipStream_t st)
{
    const int total = nch * 2 * 512;
    hipLaunchKernelGGL(repack, dim3(grid_cap(total, 256, 1024)), dim3(256), 0, st, W, cout, cin, cins, nch, dgrad,
                       lo_pairs, out);
    return hipGetLastError();
}

} // namespace nn
} // namespace gs
