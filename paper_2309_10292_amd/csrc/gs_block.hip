// Gray-Scott sweep of small grids for gfx950: T = 1..4 time steps of one block
// per workgroup, entirely in LDS (Eq. 2a/2b applied T times with the Eq. 1a/1b
// sources and the Eq. 3 Laplacian; periodic in x, y, z).
//
// A workgroup owns an output block of 4 BXG x BY x BZ cells, loads it with a
// halo of T planes and rows and one x-group (4 cells, enough for T <= 4) on
// each side into LDS, and advances the whole region level by level. Level k
// (the state after k of the T steps) is computed where it is needed: rows and
// planes k .. R - 1 - k of the region, every x-group (level T: the output block
// alone). The cells of a level are dealt to the lanes afresh, one x-group in PZ
// neighbouring planes per lane, so no lane is spent on positions a level does
// not need; levels overwrite the region in place between two barriers.
//
// What bounds it: latency. A launch of one 8x4x4 block per CU (32^3 cells, FP64)
// takes 4.3 us for one step (launch, one round of loads, one level, stores) and
// about 0.9 us for each further one: a level reads 22 values of each field per
// x-group from LDS (LDS and FP64 issue each about 0.7 CU clocks per
// cell-update, and the barriers keep them from overlapping fully). A z-streaming
// workgroup spends two barriers on every plane instead, and a launch of T = 2
// takes 8 to 10 us at any size below 64^3. Per step, FP64 without noise: 32^3
// 4.53 -> 1.72 us, 48^3 4.77 -> 2.41, 64^3 4.89 -> 3.18. Two planes per lane
// (PZ = 2) read a fifth less LDS but leave half the waves to hide a level's
// latency: 32^3 T = 4 2.00 against 1.72 us, and faster only where the blocks
// are many and shallow (80^3, 16x8x4, T = 2: 4.97 against 5.40) or one plane
// per lane needs more lanes than a workgroup has (16x8x8, T = 4).
#include "gs_device.hpp"
#include "gs_launch.hpp"
#include "gs_tblock_common.hpp"

namespace gs {

template <typename S, int BXG, int BY, int BZ, int T, int PZ> struct BlkGeom {
    typedef typename Traits<S>::C C;
    static constexpr int GX = BXG + 2, RY = BY + 2 * T, RZ = BZ + 2 * T; // region: x-groups, rows, planes
    static constexpr int PL = RY * GX;                                  // x-groups of a plane
    static constexpr int NU = PL * RZ;
    // Lanes of level k: an x-group in PZ neighbouring planes each.
    static constexpr int lanes(int k) { return k < T ? GX * (RY - 2 * k) * ((RZ - 2 * k) / PZ) : BXG * BY * (BZ / PZ); }
    static constexpr int NT = (lanes(1) + 63) / 64 * 64;
    // An x-group's 4 cells are one 16-byte vector in FP32; in FP64 they are two,
    // kept in separate arrays (halves), so that neighbouring lanes read
    // neighbouring vectors in every access.
    static constexpr int NH = sizeof(C) / 4, HC = 4 / NH; // halves, cells per half
    static constexpr int HALF = NU * HC;                  // elements of one half of one field
    static constexpr int FIELD = NH * HALF;
    static_assert(BZ % 2 == 0 && (PZ == 1 || PZ == 2), "whole lanes per column");
    static_assert(T >= 1 && T <= 4, "one halo x-group covers at most 4 levels");
    static_assert(2 * FIELD * sizeof(C) <= 160 * 1024, "the region fits the LDS of a CU");
};

__device__ __forceinline__ int wrap_any(int i, int n)
{
    while (i < 0) i += n;
    while (i >= n) i -= n;
    return i;
}

template <typename S, int BXG, int BY, int BZ, int T, int PZ, bool NOISE>
__global__ __launch_bounds__((BlkGeom<S, BXG, BY, BZ, T, PZ>::NT)) void stencil_blk(const S *__restrict__ u,
                                                                              const S *__restrict__ v,
                                                                              S *__restrict__ un, S *__restrict__ vn,
                                                                              StepArgs a)
{
    typedef BlkGeom<S, BXG, BY, BZ, T, PZ> G;
    typedef typename G::C C;
    typedef C HV __attribute__((ext_vector_type(G::HC))); // one 16-byte LDS vector
    __shared__ HV lds_v[2 * G::FIELD / G::HC];
    const C *lds = reinterpret_cast<const C *>(lds_v);
    const int tid = threadIdx.x;
    const uint32_t lb = xcd_logical_block(blockIdx.x, gridDim.x);
    const int bx = (int)(lb % (uint32_t)a.ntx);
    const uint32_t rest = lb / (uint32_t)a.ntx;
    const int x0 = bx * (4 * BXG), y0 = (int)(rest % (uint32_t)a.nty) * BY, z0 = (int)(rest / (uint32_t)a.nty) * BZ;
    const int nx = a.nx, ny = a.ny, nz = a.nz;
    const uint64_t t0 = NOISE ? step_index(a) : 0;
    const CoefF32 kf = coef_f32(a);

    // 16-byte vector of half h of x-group (xg, y, z) of field f
    auto vec_at = [&](int f, int h, int z, int y, int xg) { return ((f * G::NH + h) * G::RZ + z) * G::PL + y * G::GX + xg; };

    // This lane's x-group (xg, y, z) of level k (z: the first of its PZ planes).
    auto position = [&](int k, int &xg, int &y, int &z) {
        const int gxk = k < T ? G::GX : BXG, ryk = G::RY - 2 * k;
        xg = tid % gxk + (k < T ? 0 : 1);
        y = tid / gxk % ryk + k;
        z = tid / (gxk * ryk) * PZ + k;
    };

    // Level 0: every x-group of the region, all loads in flight together.
    uint32_t wq[NOISE ? T : 1][PZ][4];
    constexpr int ROUNDS = (G::NU + G::NT - 1) / G::NT;
    {
        Vec<S, 4> q[ROUNDS][2];
#pragma unroll
        for (int r = 0; r < ROUNDS; ++r) {
            const int p = min(tid + r * G::NT, G::NU - 1);
            const int xg = p % G::GX, y = p / G::GX % G::RY, z = p / G::PL;
            const size_t off = (size_t)wrap_any(x0 - 4 + 4 * xg, nx) +
                               (size_t)nx * ((size_t)wrap_any(y0 - T + y, ny) + (size_t)ny * wrap_any(z0 - T + z, nz));
            q[r][0] = *reinterpret_cast<const Vec<S, 4> *>(u + off);
            q[r][1] = *reinterpret_cast<const Vec<S, 4> *>(v + off);
        }
        // the noise of every level, made while the loads are on their way
        if constexpr (NOISE) {
#pragma unroll
            for (int k = 1; k <= T; ++k) {
                int xg, y, z;
                position(k, xg, y, z);
                const size_t row = (size_t)wrap_any(x0 - 4 + 4 * xg, nx) + (size_t)nx * wrap_any(y0 - T + y, ny);
#pragma unroll
                for (int j = 0; j < PZ; ++j) {
                    const size_t idx = row + (size_t)nx * ny * wrap_any(z0 - T + z + j, nz);
                    const Philox4 w = noise_block(idx, t0 + (uint64_t)(k - 1), a.seed);
#pragma unroll
                    for (int e = 0; e < 4; ++e) wq[k - 1][j][e] = w.w[e];
                }
            }
        }
#pragma unroll
        for (int r = 0; r < ROUNDS; ++r) {
            const int p = min(tid + r * G::NT, G::NU - 1);
#pragma unroll
            for (int f = 0; f < 2; ++f)
#pragma unroll
                for (int h = 0; h < G::NH; ++h) {
                    HV w;
#pragma unroll
                    for (int e = 0; e < G::HC; ++e) w[e] = fload<S>(f, q[r][f].e[h * G::HC + e]);
                    lds_v[(f * G::NH + h) * G::NU + p] = w;
                }
        }
    }
    __syncthreads();

    auto level = [&](auto lev) {
        constexpr int k = decltype(lev)::value;
        constexpr bool LAST = k == T;
        const bool act = tid < G::lanes(k);
        C res[PZ][2][4]; // [plane][field][cell]
        int xg, y, z;
        position(k, xg, y, z);
        if (act) {
            C c[2][PZ + 2][4], lap[PZ][2][4]; // centre column with its z neighbours, Laplacians
#pragma unroll
            for (int f = 0; f < 2; ++f) {
                auto group = [&](int zz, int yy, C (&o)[4]) {
#pragma unroll
                    for (int h = 0; h < G::NH; ++h) {
                        const HV w = lds_v[vec_at(f, h, zz, yy, xg)];
#pragma unroll
                        for (int e = 0; e < G::HC; ++e) o[h * G::HC + e] = w[e];
                    }
                };
#pragma unroll
                for (int j = 0; j < PZ + 2; ++j) group(z - 1 + j, y, c[f][j]);
#pragma unroll
                for (int j = 0; j < PZ; ++j) {
                    C ym[4], yp[4];
                    group(z + j, y - 1, ym);
                    group(z + j, y + 1, yp);
                    // x-edges: the last cell of the group before, the first of the one after
                    const C xl = lds[vec_at(f, G::NH - 1, z + j, y, xg - 1) * G::HC + G::HC - 1];
                    const C xr = lds[vec_at(f, 0, z + j, y, xg + 1) * G::HC];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const C cc = c[f][j + 1][e];
                        const C xm = e > 0 ? c[f][j + 1][e > 0 ? e - 1 : 0] : xl, xp = e < 3 ? c[f][j + 1][e < 3 ? e + 1 : 3] : xr;
                        if constexpr (sizeof(C) == 8)
                            lap[j][f][e] = lap_f64(cc, xm, xp, ym[e], yp[e], c[f][j][e], c[f][j + 2][e]);
                        else
                            lap[j][f][e] = lap6_f32<S>(cc, xm, xp, ym[e], yp[e], c[f][j][e], c[f][j + 2][e]);
                    }
                }
            }
#pragma unroll
            for (int j = 0; j < PZ; ++j) {
                C r[4] = {(C)0, (C)0, (C)0, (C)0};
                if constexpr (NOISE) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        if constexpr (sizeof(C) == 8)
                            r[e] = __builtin_fma(a.noise_s, (double)(int32_t)wq[k - 1][j][e], a.noise_h);
                        else
                            r[e] = noise_term_f32(wq[k - 1][j][e], kf.ns, kf.nh);
                    }
                }
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    C uo, vo;
                    // dt = 1 needs no variant: the products are exact
                    cell_update<C, false, NOISE>(a, kf, c[0][j + 1][e], c[1][j + 1][e], lap[j][0][e], lap[j][1][e], r[e], uo, vo);
                    res[j][0][e] = fload<S>(0, fstore<S>(0, uo));
                    res[j][1][e] = fload<S>(1, fstore<S>(1, vo));
                }
            }
        }
        if constexpr (LAST) {
            const int x = x0 + 4 * (xg - 1), yy = y0 + y - T, zz = z0 + z - T;
            if (act && x < nx && yy < ny) {
#pragma unroll
                for (int j = 0; j < PZ; ++j)
                    if (zz + j < nz) {
                        const size_t off = (size_t)x + (size_t)nx * ((size_t)yy + (size_t)ny * (zz + j));
                        Vec<S, 4> ou, ov;
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            ou.e[e] = fstore<S>(0, res[j][0][e]);
                            ov.e[e] = fstore<S>(1, res[j][1][e]);
                        }
                        *reinterpret_cast<Vec<S, 4> *>(un + off) = ou;
                        *reinterpret_cast<Vec<S, 4> *>(vn + off) = ov;
                    }
            }
        } else {
            __syncthreads(); // every read of level k-1 is done
            if (act) {
#pragma unroll
                for (int j = 0; j < PZ; ++j)
#pragma unroll
                    for (int f = 0; f < 2; ++f)
#pragma unroll
                        for (int h = 0; h < G::NH; ++h) {
                            HV w;
#pragma unroll
                            for (int e = 0; e < G::HC; ++e) w[e] = res[j][f][h * G::HC + e];
                            lds_v[vec_at(f, h, z + j, y, xg)] = w;
                        }
            }
            __syncthreads();
        }
    };
    level(Phase<1>{});
    if constexpr (T >= 2) level(Phase<2>{});
    if constexpr (T >= 3) level(Phase<3>{});
    if constexpr (T >= 4) level(Phase<4>{});
}

// ------------------------------------------------------------------ launch
template <typename S, int BXG, int BY, int BZ, int T, int PZ>
static hipError_t launch_blk_t(const void *u, const void *v, void *un, void *vn, StepArgs a, hipStream_t st)
{
    a.ntx = (a.nx + 4 * BXG - 1) / (4 * BXG);
    a.nty = (a.ny + BY - 1) / BY;
    const size_t nb = (size_t)a.ntx * a.nty * ((a.nz + BZ - 1) / BZ);
    const int nt = BlkGeom<S, BXG, BY, BZ, T, PZ>::NT;
    if (!grid_fits(nb, nt)) return hipErrorInvalidConfiguration;
    if (a.noise != 0.0)
        hipLaunchKernelGGL((stencil_blk<S, BXG, BY, BZ, T, PZ, true>), dim3((unsigned)nb), dim3(nt), 0, st, (const S *)u,
                           (const S *)v, (S *)un, (S *)vn, a);
    else
        hipLaunchKernelGGL((stencil_blk<S, BXG, BY, BZ, T, PZ, false>), dim3((unsigned)nb), dim3(nt), 0, st, (const S *)u,
                           (const S *)v, (S *)un, (S *)vn, a);
    return hipGetLastError();
}

int num_blk_shapes() { return 3; }

BlkShape blk_shape(int shape)
{
    switch (shape) {
    case 1: return BlkShape{8, 4, 4};
    case 2: return BlkShape{16, 8, 4};
    case 3: return BlkShape{16, 8, 8};
    }
    return BlkShape{0, 0, 0};
}

template <typename S, int T>
static hipError_t blk_dispatch_shape(int shape, const void *u, const void *v, void *un, void *vn, const StepArgs &a,
                                     hipStream_t st)
{
    switch (shape) {
    case 1: return launch_blk_t<S, 2, 4, 4, T, 1>(u, v, un, vn, a, st);
    case 2: return launch_blk_t<S, 4, 8, 4, T, T <= 2 ? 2 : 1>(u, v, un, vn, a, st);
    case 3: return launch_blk_t<S, 4, 8, 8, T, T == 4 ? 2 : 1>(u, v, un, vn, a, st);
    }
    return hipErrorInvalidValue;
}

template <typename S>
static hipError_t blk_dispatch(int T, int shape, const void *u, const void *v, void *un, void *vn, const StepArgs &a,
                               hipStream_t st)
{
    switch (T) {
    case 1: return blk_dispatch_shape<S, 1>(shape, u, v, un, vn, a, st);
    case 2: return blk_dispatch_shape<S, 2>(shape, u, v, un, vn, a, st);
    case 3: return blk_dispatch_shape<S, 3>(shape, u, v, un, vn, a, st);
    case 4: return blk_dispatch_shape<S, 4>(shape, u, v, un, vn, a, st);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_block(int storage, int T, int shape, const void *u, const void *v, void *un, void *vn,
                        const StepArgs &a, hipStream_t st)
{
    switch (storage) {
    case 0: return blk_dispatch<double>(T, shape, u, v, un, vn, a, st);
    case 1: return blk_dispatch<float>(T, shape, u, v, un, vn, a, st);
    case 2: return blk_dispatch<bf16>(T, shape, u, v, un, vn, a, st);
    case 3: return blk_dispatch<f16>(T, shape, u, v, un, vn, a, st);
    case 4: return blk_dispatch<bf16c>(T, shape, u, v, un, vn, a, st);
    }
    return hipErrorInvalidValue;
}

} // namespace gs
