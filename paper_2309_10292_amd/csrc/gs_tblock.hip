// Temporally blocked Gray-Scott sweep for gfx950: T = 1..4 time steps per
// pass over HBM (Eq. 2a/2b applied T times with the Eq. 1a/1b sources and the
// Eq. 3 Laplacian; periodic in x, y, z).
//
// One workgroup of NT lanes owns an output tile of TXG x-groups (4 cells
// each) by TY rows and marches through a chunk of z planes. Level k (k = 0..T)
// is the state after k of the T steps; level k is needed on the output tile
// widened by T - k rows in y and by one x-group on each side in x (enough for
// T <= 4). Every lane owns one x-group of the level-0 region and the same
// position in every level. The depth of a position is the last level that
// needs it; lanes are ordered by decreasing depth, so a wave whose positions
// are all shallower than level k skips level k as a whole.
//
// Per z iteration i (a wavefront in z):
//   - level-0 plane i+1 enters (prefetched one iteration earlier, into
//     registers or, in the FP64 kernel with noise at three fused steps,
//     straight into a lane-private LDS area);
//   - for k = 1..T, level k computes plane i-k+1 from level k-1's planes
//     i-k, i-k+1, i-k+2: z neighbours from the lane's registers (three plane
//     slots per level; plane z sits in slot (z - i0) mod 3, and the loop is
//     unrolled by three so that slots are fixed registers), x and y neighbours
//     from level k-1's current plane staged in LDS;
//   - level T's plane is stored if it lies in the workgroup's chunk;
//   - each level's newest plane is staged in LDS for the next iteration.
// Every cell-update rounds exactly as the single-step kernel's (the same
// operation sequence; in FP64 the noise term n r is one fused operation on the
// same exact real), so results are bitwise independent of T and of the tile.
// The noise of level k uses step index t + k - 1.
#include "gs_device.hpp"
#include "gs_launch.hpp"
#include "gs_tblock_common.hpp"

namespace gs {

// The FP64 kernel with noise at three fused steps and 512 lanes prefetches
// level 0 through LDS (global_load_lds, 16 bytes per lane and load) instead
// of registers, and makes the next iteration's Philox blocks between the two
// barriers of an iteration, where the vector units otherwise wait for the
// LDS stores: the registers this frees keep its straight-line levels free of
// spills.
template <typename S, int T, int NT, int NOISE> constexpr bool tb_dma()
{
    return sizeof(S) == 8 && NOISE && T == 3 && NT == 512;
}
// FP64 kernels whose noise has 64-bit block indices on every grid: those that the
// registers bind most, where the 32-bit ones' few more cost spills or their places (320 x
// 320 x 256 with noise, chunks of 4 planes, us per step: 1024 lanes 222 -> 203, 768
// lanes at two steps 142 -> 137, 512 lanes at four 232 -> 217; 512 lanes at three,
// chunks of 16, keep the 32-bit ones, 107 against 111).
// FP32's three steps in 1024 lanes spill nothing then (14 otherwise), and its single step
// in 768 takes the 80 registers that let two workgroups share a CU.
template <typename S, int T, int NT> constexpr bool tb_noise_64()
{
    return sizeof(S) == 8   ? NT > 512 || (NT == 512 && T == 4)
           : sizeof(S) == 4 ? (NT == 768 && T == 1) || (NT == 1024 && T == 3)
                            : false;
}
// FP32 kernels whose coefficients stay in scalar registers: those of 768 and 1024 lanes,
// where vector ones made them spill (three steps in 1024 lanes, 320 x 320 x 256 with
// noise, chunks of 16 planes: 102 -> 86 us per step; without noise 67.7 -> 65.8) or lose
// a workgroup per CU (one step in 768 lanes with noise, chunks of 4: 108 -> 94).
template <typename S, int NT> constexpr bool tb_coef_scalar() { return sizeof(S) == 4 && NT > 512; }
// Complemented BF16 without noise: the kernels that round a cell as soon as it is done
// instead of all four in pairs. The paired rounding takes fewer instructions, and longer
// where one workgroup of 768 or 1024 lanes fills a CU or 512 lanes keep four levels (320 x
// 320 x 256, chunks of 16 planes, us per step: 768 lanes 52.5 -> 48.4 at two steps and
// 53.6 -> 48.9 at three, 1024 lanes 56.2 -> 54.3 and 61.8 -> 58.0, 128-cell tile at four
// 131 -> 116; 256 lanes at four would lose a fifth).
template <typename S, int T, int NT, int NOISE> constexpr bool tb_round_cells()
{
    return Complemented<S>::value && !NOISE && T >= 2 && (NT > 512 || (NT == 512 && T == 4));
}
// A workgroup barrier that waits for the LDS operations only: the LDS-DMA
// prefetch stays in flight across it (each wave reads only the area its own
// loads fill, after waiting for them).
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_s_waitcnt(0xC07F); // lgkmcnt(0)
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    __builtin_amdgcn_s_barrier();
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
}

template <typename S, int TXG, int TY, int T, int NT> struct TbGeom {
    typedef typename Traits<S>::C C;
    static constexpr int GX = TXG + 2;          // x-groups per region row
    static constexpr int RW = GX * 4;           // region row width (cells)
    static constexpr int H = 16 / (int)sizeof(C);  // LDS row pad (>= 1; keeps rows 16-byte aligned)
    static constexpr int RY0 = TY + 2 * T;      // level-0 rows
    static constexpr int NSLOT = GX * RY0;      // lanes with a level-0 position
    // LDS rows of levels 0..T-1: RY0 - 2k each.
    static constexpr int LDS_ROWS = T * RY0 - T * (T - 1);
    // FP64 rows are split in two half-rows: cells 0-1 of every x-group, then
    // cells 2-3. A lane's four cells are 32 bytes, and 16-byte LDS accesses at
    // a 32-byte lane stride conflict in the banks; in half-rows every 16-byte
    // access of a row of lanes is contiguous. Each half-row has a pad group on
    // either side for the x-neighbours at the region's edges. FP32 rows (16
    // bytes per lane) are contiguous as they are.
    static constexpr bool SPLIT = sizeof(C) == 8;
    static constexpr int HS = 2 * (GX + 2);     // half-row length
    static constexpr int RS_MIN = SPLIT ? 2 * HS : RW + 2 * H;
    // A wave holds several rows of TXG lanes; their 16-byte reads are free of bank
    // conflicts on gfx950 only when each row goes on where the one before ends,
    // modulo 256 bytes (measured with the LDS counters for 16 lanes: 640- and
    // 320-byte strides conflict two ways). Rows are padded to that where the padded
    // planes (and the FP64 kernel's prefetch area) fit the LDS of a CU.
    static constexpr int RS_MIN_B = RS_MIN * (int)sizeof(C);
    static constexpr int RS_PAD_B = RS_MIN_B + (TXG * 16 - RS_MIN_B % 256 + 512) % 256;
    static constexpr int DMA_B = SPLIT && T == 3 && NT == 512 ? 4 * NT * 16 : 0;
    static constexpr int RS = (2 * LDS_ROWS * RS_PAD_B + DMA_B <= 160 * 1024 ? RS_PAD_B : RS_MIN_B) / (int)sizeof(C); // row stride
    // Offset within a row of column 4 gx + e of the region (e = -1 .. 4):
    // a per-lane base plus a constant, so every access of a lane shares one
    // address register.
    static __host__ __device__ constexpr int lane_base(int gx) { return SPLIT ? 2 * (gx + 1) : H + 4 * gx; }
    static __host__ __device__ constexpr int cell_off(int e)
    {
        return SPLIT ? (e < 0 ? HS - 1 : e < 2 ? e : e < 4 ? HS + e - 2 : 2) : e;
    }
    static constexpr int FIELD = LDS_ROWS * RS; // elements per field
    static_assert(T >= 1 && T <= 4, "one pad group covers at most 4 levels");
    static_assert(NSLOT <= NT, "every level-0 position needs a lane");
    static_assert(2 * FIELD * sizeof(C) <= 160 * 1024, "staged planes fit the LDS of a CU");
    static constexpr int row_base(int k) { return k * RY0 - k * (k - 1); }
};

// One output tile [x0, x0 + 4 TXG) x [y0, y0 + TY) x [z0, ze) of a grid
// (a.nx, a.ny, a.nz), T steps from (u, v) into (un, vn); t0 is the step index
// of the first of the T steps. `lds` holds 2 * TbGeom::FIELD elements and
// `pre_lds` 4 * NT 16-byte slots where tb_dma() holds (else it is unused).
// Every lane of the workgroup must call it (it contains barriers).
template <typename S, int TXG, int TY, int T, int NT, int NOISE, bool UNIT_DT, bool LINE>
__device__ __forceinline__ void tb_tile(const S *__restrict__ u, const S *__restrict__ v, S *__restrict__ un,
                                        S *__restrict__ vn, const StepArgs &a, int x0, int y0, int z0, int ze,
                                        uint64_t t0, typename Traits<S>::C *__restrict__ lds,
                                        uint4 *__restrict__ pre_lds)
{
    typedef TbGeom<S, TXG, TY, T, NT> G;
    typedef typename G::C C;
    constexpr bool DMA = tb_dma<S, T, NT, NOISE>();
    constexpr bool CELLS = tb_round_cells<S, T, NT, NOISE>();
    static_assert(!DMA || 2 * G::FIELD * sizeof(C) + 4 * NT * 16 <= 160 * 1024, "staged planes and prefetch fit");
    const int nx = a.nx, ny = a.ny, nz = a.nz;
    const size_t plane = (size_t)nx * (size_t)ny;
    const CoefF32 kf = tb_coef_scalar<S, NT>() ? coef_f32_scalar(a) : coef_f32(a);

    // This lane's position (x-group gxs, level-0 row rys) and depth dep
    // (-1: none). Order: the output tile (depth T, row-major), the x-halo
    // groups beside the output rows (depth T-1), then rows d and RY0-1-d for
    // d = T-1 down to 0 (depth d).
    int gxs = 0, rys = 0, dep = -1;
    {
        constexpr int nA = TXG * TY, nH = 2 * TY;
        const int s = threadIdx.x;
        if (s < nA) {
            rys = T + s / TXG;
            gxs = 1 + s % TXG;
            dep = T;
        } else if (s < nA + nH) {
            const int r = s - nA;
            rys = T + (r >> 1);
            gxs = (r & 1) ? G::GX - 1 : 0;
            dep = T - 1;
        } else {
            const int r = s - nA - nH;
            const int d = T - 1 - r / (2 * G::GX);
            if (d >= 0) {
                const int q = r % (2 * G::GX);
                rys = q < G::GX ? d : G::RY0 - 1 - d;
                gxs = q % G::GX;
                dep = d;
            }
        }
    }
    const bool has = dep >= 0;
    const int gx = (((x0 - 4 + 4 * gxs) % nx) + nx) % nx;
    const int gy = (((y0 - T + rys) % ny) + ny) % ny;
    const size_t xy = (size_t)gy * nx + gx;
    // Output positions are exactly the depth-T ones.
    const bool out_ok = dep == T && (x0 + 4 * (gxs - 1) < nx) && (y0 + rys - T < ny);

    C win[T][3][2][4]; // [level][slot][field][cell]
#pragma unroll
    for (int k = 0; k < T; ++k)
#pragma unroll
        for (int q = 0; q < 3; ++q)
#pragma unroll
            for (int f = 0; f < 2; ++f)
#pragma unroll
                for (int e = 0; e < 4; ++e) win[k][q][f][e] = (C)0;

    const S *src[2] = {u, v};
    auto load_plane = [&](int z, Vec<S, 4> (&o)[2]) {
        const size_t off = (size_t)wrap(z, nz) * plane + xy;
#pragma unroll
        for (int f = 0; f < 2; ++f) o[f] = *reinterpret_cast<const Vec<S, 4> *>(src[f] + off);
    };
    const int lbase = G::lane_base(gxs);
    // Element e (-1 .. 4, column 4 gxs + e) of row `row` of level k's plane.
    auto lds_at = [&](int f, int k, int row, int e) -> C & {
        return lds[f * G::FIELD + (G::row_base(k) + row) * G::RS + lbase + G::cell_off(e)];
    };
    auto in_level = [&](int k) { return dep >= k; };

    // LDS-DMA prefetch (tb_dma): slot 2 f + hh of a lane holds cells
    // 2 hh, 2 hh + 1 of field f; a wave's 64 lanes fill 64 consecutive slots.
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    auto dma_plane = [&](int z) {
        const size_t off = (size_t)wrap(z, nz) * plane + xy;
#pragma unroll
        for (int f = 0; f < 2; ++f)
#pragma unroll
            for (int hh = 0; hh < 2; ++hh)
                __builtin_amdgcn_global_load_lds((const void *)(src[f] + off + 2 * hh),
                                                 (__attribute__((address_space(3))) void *)(pre_lds + (2 * f + hh) * NT +
                                                                                            64 * wave),
                                                 16, 0, 0);
    };
    auto read_pre = [&](C (&o)[2][4]) {
#pragma unroll
        for (int f = 0; f < 2; ++f)
#pragma unroll
            for (int hh = 0; hh < 2; ++hh) {
                const double2 q = *reinterpret_cast<const double2 *>(pre_lds + (2 * f + hh) * NT + threadIdx.x);
                o[f][2 * hh] = q.x;
                o[f][2 * hh + 1] = q.y;
            }
    };
    // The noise block of this lane's position in plane z at level k.
    const uint32_t xyq = (uint32_t)(xy >> 2), planeq = (uint32_t)(plane >> 2);
    auto noise_at = [&](int z, int k) {
        if constexpr (NOISE == NOISE_32) return noise_block32((uint32_t)z * planeq + xyq, t0 + (uint64_t)(k - 1), a.seed);
        else return noise_block((size_t)z * plane + xy, t0 + (uint64_t)(k - 1), a.seed);
    };
    // Philox blocks of the next iteration's levels (tb_dma), made ahead.
    uint32_t wq[T][4];
    auto make_noise = [&](const int i, auto full) {
        constexpr bool FULL = decltype(full)::value;
#pragma unroll
        for (int k = 1; k <= T; ++k) {
            if (!FULL && !in_level(k)) continue;
            const Philox4 w = noise_at(wrap(i - k + 1, nz), k);
#pragma unroll
            for (int e = 0; e < 4; ++e) wq[k - 1][e] = w.w[e];
        }
    };

    // Prologue: level-0 slots hold planes i0-1 (slot 2) and i0 (slot 0); plane
    // i0+1 is in flight; LDS holds level-0 plane i0.
    const int i0 = z0 - T + 1;
    const int i_end = ze + T - 2; // inclusive
    Vec<S, 4> pre[2];
    if constexpr (DMA) dma_plane(i0 + 1);
    if (has) {
        Vec<S, 4> q0[2], q1[2];
        load_plane(i0 - 1, q0);
        load_plane(i0, q1);
        if constexpr (!DMA) load_plane(i0 + 1, pre);
#pragma unroll
        for (int f = 0; f < 2; ++f)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                win[0][2][f][e] = fload<S>(f, q0[f].e[e]);
                win[0][0][f][e] = fload<S>(f, q1[f].e[e]);
            }
#pragma unroll
        for (int f = 0; f < 2; ++f)
#pragma unroll
            for (int e = 0; e < 4; ++e) lds_at(f, 0, rys, e) = win[0][0][f][e];
    }
    if constexpr (DMA) {
        make_noise(i0, Full<true>{});
        lds_barrier();
    } else {
        __syncthreads();
    }

    // One z iteration at phase P = (i - i0) mod 3. A wave whose first lane
    // (the deepest position of the wave) has depth T runs every level on all
    // of its lanes without per-lane branches (FULL): the lanes that a level
    // does not need compute values nobody reads, from clamped LDS rows, and
    // only the stores stay per-lane. Straight-line levels let the scheduler
    // overlap the Philox chains with LDS reads and arithmetic. Other waves
    // skip, per lane, the levels their positions do not need.
    auto iteration = [&](const int i, auto phase, auto full) {
        constexpr int P = decltype(phase)::value;
        constexpr bool FULL = decltype(full)::value;
        // Level 0: plane i+1 enters its slot; prefetch plane i+2.
        if constexpr (DMA) {
            __builtin_amdgcn_s_waitcnt(0x0F70); // vmcnt(0): this wave's prefetch has landed
            read_pre(win[0][slot3(P + 1)]);
            __builtin_amdgcn_s_waitcnt(0xC07F); // lgkmcnt(0): read before it is overwritten
            if (i + 2 <= ze + T - 1) dma_plane(i + 2);
        } else {
#pragma unroll
            for (int f = 0; f < 2; ++f)
#pragma unroll
                for (int e = 0; e < 4; ++e) win[0][slot3(P + 1)][f][e] = fload<S>(f, pre[f].e[e]);
            if (has && i + 2 <= ze + T - 1) load_plane(i + 2, pre);
        }

        // Levels 1..T, in order; level k computes plane i-k+1.
#pragma unroll
        for (int k = 1; k <= T; ++k) {
            if (!FULL && !in_level(k)) continue;
            const int zk = i - k + 1;
            const int sm = slot3(P - k), sc = slot3(P - k + 1), sp = slot3(P - k + 2);
            // Row of this position in level k-1's LDS plane (clamped for
            // positions outside level k, whose results are not used).
            const int ry = FULL ? min(max(rys, k), G::RY0 - 1 - k) : rys;
            const int row = ry - (k - 1);
            C xm[2][4], xp[2][4], ym[2][4], yp[2][4];
#pragma unroll
            for (int f = 0; f < 2; ++f) {
                const C *c = win[k - 1][sc][f];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    xm[f][e] = e > 0 ? c[e - 1] : lds_at(f, k - 1, row, -1);
                    xp[f][e] = e < 3 ? c[e + 1] : lds_at(f, k - 1, row, 4);
                    ym[f][e] = lds_at(f, k - 1, row - 1, e);
                    yp[f][e] = lds_at(f, k - 1, row + 1, e);
                }
            }
            C r[4] = {(C)0, (C)0, (C)0, (C)0}; // the noise term n r
            if constexpr (NOISE) {
                Philox4 w;
                if constexpr (DMA) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) w.w[e] = wq[k - 1][e];
                } else {
                    w = noise_at(wrap(zk, nz), k);
                }
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    // FP64: n r with r = (w + 1/2) 2^-31 is the exact real
                    // (n 2^-31) w + n 2^-32, so one fused operation rounds it
                    // once, as the product n r does.
                    if constexpr (sizeof(C) == 8)
                        r[e] = __builtin_fma(a.noise_s, (double)(int32_t)w.w[e], a.noise_h);
                    else
                        r[e] = noise_term_f32(w.w[e], kf.ns, kf.nh);
                }
            }
            C res[2][4];
            C lap[2][4]; // FP64: the Laplacians; FP32: six times them
            if constexpr (sizeof(C) == 4) {
#pragma unroll
                for (int f = 0; f < 2; ++f) {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        lap[f][e] = lap6_f32<S>(win[k - 1][sc][f][e], xm[f][e], xp[f][e], ym[f][e], yp[f][e],
                                                win[k - 1][sm][f][e], win[k - 1][sp][f][e]);
                }
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const C uc = win[k - 1][sc][0][e], vc = win[k - 1][sc][1][e];
                if constexpr (sizeof(C) == 8) {
                    lap[0][e] = lap_f64(uc, xm[0][e], xp[0][e], ym[0][e], yp[0][e], win[k - 1][sm][0][e], win[k - 1][sp][0][e]);
                    lap[1][e] = lap_f64(vc, xm[1][e], xp[1][e], ym[1][e], yp[1][e], win[k - 1][sm][1][e], win[k - 1][sp][1][e]);
                }
                C uo, vo;
                cell_update<C, UNIT_DT, NOISE != 0>(a, kf, uc, vc, lap[0][e], lap[1][e], r[e], uo, vo);
                res[0][e] = CELLS ? fload<S>(0, fstore<S>(0, uo)) : uo;
                res[1][e] = CELLS ? fload<S>(1, fstore<S>(1, vo)) : vo;
            }
            // Every level carries the stored precision of the state.
            Vec<S, 4> st[2];
#pragma unroll
            for (int f = 0; f < 2; ++f) {
                if constexpr (CELLS) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) st[f].e[e] = fstore<S>(f, res[f][e]); // exact
                } else {
                    st[f] = fstore4<S>(f, res[f]);
                }
            }
            if (k < T) {
#pragma unroll
                for (int f = 0; f < 2; ++f)
#pragma unroll
                    for (int e = 0; e < 4; ++e) win[k][sc][f][e] = CELLS ? res[f][e] : fload<S>(f, st[f].e[e]);
            } else if (out_ok && zk >= z0) {
                const size_t off = (size_t)zk * plane + xy;
                NtStore<S>::put(un + off, st[0]);
                NtStore<S>::put(vn + off, st[1]);
            }
        }
        if constexpr (DMA) lds_barrier(); // all reads of the staged planes are done
        else __syncthreads();
        // Stage the newest plane of levels 0..T-1 (the centre plane of the next iteration).
        if (has) {
#pragma unroll
            for (int f = 0; f < 2; ++f)
#pragma unroll
                for (int e = 0; e < 4; ++e) lds_at(f, 0, rys, e) = win[0][slot3(P + 1)][f][e];
        }
#pragma unroll
        for (int k = 1; k < T; ++k) {
            if (in_level(k)) {
#pragma unroll
                for (int f = 0; f < 2; ++f)
#pragma unroll
                    for (int e = 0; e < 4; ++e) lds_at(f, k, rys - k, e) = win[k][slot3(P - k + 1)][f][e];
            }
        }
        if constexpr (DMA) {
            make_noise(i + 1, full);
            lds_barrier();
        } else {
            __syncthreads();
        }
    };

    // The straight-line variant (LINE: not ruled out by the caller) needs more
    // registers; it is used where they fit the budget (up to 512 lanes; FP64 up to 3 levels; not FP32 storage,
    // whose FP64 sums would spill 40 registers at two levels in 128: 530 against
    // 272 us per step at 512^3 with noise).
    constexpr bool full_ok = LINE && NT <= 512 && (sizeof(S) == 2 || (sizeof(S) == 8 && T <= 3));
    const int wave_depth = __builtin_amdgcn_readfirstlane(dep);
    if (full_ok && wave_depth == T) {
        for (int i = i0; i <= i_end; i += 3) {
            iteration(i, Phase<0>{}, Full<true>{});
            if (i + 1 <= i_end) iteration(i + 1, Phase<1>{}, Full<true>{});
            if (i + 2 <= i_end) iteration(i + 2, Phase<2>{}, Full<true>{});
        }
    } else {
        for (int i = i0; i <= i_end; i += 3) {
            iteration(i, Phase<0>{}, Full<false>{});
            if (i + 1 <= i_end) iteration(i + 1, Phase<1>{}, Full<false>{});
            if (i + 2 <= i_end) iteration(i + 2, Phase<2>{}, Full<false>{});
        }
    }
}

// Waves per SIMD the single-grid kernel is compiled for (its register
// budget): with FP32 arithmetic and up to two fused steps the kernel fits 128
// registers, so 256- and 512-lane workgroups keep four waves per SIMD (two
// 512-lane workgroups per CU; one register more would leave one); other
// kernels take what their lane count allows.
template <typename S, int T, int NT> constexpr int tb_min_waves()
{
    return (sizeof(typename Traits<S>::C) == 4 && T <= 2 && NT <= 512) ? 4 : 1;
}

// The output tile (bx, by) and chunk bz of the grid in `a` by this workgroup;
// `lds` and `pre_lds` as tb_tile takes them.
template <typename S, int TXG, int TY, int T, int NT, int NOISE, bool LINE = true>
__device__ __forceinline__ void tb_item(const S *__restrict__ u, const S *__restrict__ v, S *__restrict__ un,
                                        S *__restrict__ vn, const StepArgs &a, int bx, int by, int bz, uint64_t t0,
                                        typename Traits<S>::C *lds, uint4 *pre_lds)
{
    const int z0 = bz * a.zc, ze = min(z0 + a.zc, a.nz);
    // FP64 runs with dt = 1 (the workload of the paper) take the variant
    // without the dt products.
    if constexpr (sizeof(S) == 8) {
        if (a.dt == 1.0) {
            tb_tile<S, TXG, TY, T, NT, NOISE, true, LINE>(u, v, un, vn, a, bx * (TXG * 4), by * TY, z0, ze, t0, lds,
                                                          pre_lds);
            return;
        }
    }
    tb_tile<S, TXG, TY, T, NT, NOISE, false, LINE>(u, v, un, vn, a, bx * (TXG * 4), by * TY, z0, ze, t0, lds, pre_lds);
}

// LDS-DMA prefetch area of a workgroup (tb_dma), in 16-byte slots.
template <typename S, int T, int NT, int NOISE> constexpr int tb_pre_slots() { return tb_dma<S, T, NT, NOISE>() ? 4 * NT : 1; }

template <typename S, int TXG, int TY, int T, int NT, int NOISE>
__global__ __launch_bounds__(NT, (tb_min_waves<S, T, NT>())) void stencil_tb(const S *__restrict__ u,
                                                                           const S *__restrict__ v,
                                                                           S *__restrict__ un, S *__restrict__ vn,
                                                                           StepArgs a)
{
    __shared__ typename Traits<S>::C lds[2 * TbGeom<S, TXG, TY, T, NT>::FIELD];
    __shared__ uint4 pre_lds[tb_pre_slots<S, T, NT, NOISE>()];
    const uint32_t lb = xcd_logical_block(blockIdx.x, gridDim.x);
    const uint32_t rest = lb / (uint32_t)a.ntx;
    tb_item<S, TXG, TY, T, NT, NOISE>(u, v, un, vn, a, (int)(lb % (uint32_t)a.ntx), (int)(rest % (uint32_t)a.nty),
                                      (int)(rest / (uint32_t)a.nty), NOISE ? step_index(a) : 0, lds, pre_lds);
}

// The shapes: a workgroup of `lanes` lanes takes output tiles of 4 txg cells by
// rows - 2 T rows at T fused steps, from a level-0 region of (txg + 2) x-groups by
// `rows` rows. 6 and 7 are for rows that 64 cells cover badly: single grids of one to
// three steps, and the items of shape 2's batches that the host gives their width.
struct TbDef {
    int txg, rows, lanes;
};
constexpr int k_tb_shapes = 5, k_tb_narrow = 2, k_tb_depth = 4;
constexpr TbDef tb_def(int shape)
{
    constexpr TbDef d[k_tb_shapes + k_tb_narrow] = {{16, 14, 256},  {16, 28, 512}, {32, 14, 512}, {16, 42, 768},
                                                    {16, 56, 1024}, {8, 51, 512},  {12, 36, 512}};
    return d[shape - 1];
}
// One workgroup per CU: NT lanes leave 512 / ceil(NT / 256) registers per lane. The
// deepest fusion whose registers fit that budget (FP64 at four steps spills some tens);
// batched sweeps take the larger shapes one step less deep; 0: not available.
template <typename S, bool BATCH> constexpr int tb_max_T_shape(int shape)
{
    if (shape > k_tb_shapes) return BATCH ? 0 : 3;
    const int lanes = tb_def(shape).lanes;
    if (lanes <= 512) return 4;
    if (lanes <= 768) return sizeof(S) == 8 ? (BATCH ? 1 : 2) : (BATCH ? 3 : 4);
    return sizeof(S) == 8 ? (BATCH ? 0 : 1) : (BATCH ? 2 : 3);
}

// The kernel whose launches of more workgroups than are resident do without straight-line
// levels: FP64 without noise at three steps in 256 lanes takes 283 registers with them,
// which let one workgroup into a CU, and 220 without, two (16 grids of 128^3 in chunks of
// 64 planes: 143 us per step with them, 111 without; 256 items, all resident: 8.3 with
// them, 9.1 without).
template <typename S, int T, int NT, int NOISE> constexpr bool tb_packs()
{
    return sizeof(S) == 8 && T == 3 && NT == 256 && NOISE == NOISE_OFF;
}

// Sweep over many independent simulations: one workgroup per work item (one
// tile x z-chunk of one simulation), items sorted by decreasing cost, so that
// the places that fall free last are filled with the cheapest ones. Items are
// dealt to the XCDs in ranges of `slots` (about what is resident at once):
// neighbouring tiles on one XCD, and every XCD long and short items. WIDTHS: an item
// of the 64-cell shape of 512 lanes may be of the narrow shapes' tiles instead (the
// host picks a grid's width), so that one launch covers grids of 80 cells with six
// tiles and grids of 128 with twelve: 32 grids of 32^3 to 192^3 in FP64, 12 steps,
// 2.18 -> 2.03 ms. A launch without such items takes the kernel without them (32 x
// 128^3 FP32 with it: 1.97 -> 2.00 ms). PACKED: without straight-line levels (tb_packs).
enum { BATCH_PLAIN = 0, BATCH_WIDTHS = 1, BATCH_PACKED = 2 };
template <typename S, int TXG, int TY, int T, int NT, int NOISE, int FORM>
__global__ __launch_bounds__(NT, (tb_min_waves<S, T, NT>())) void stencil_tb_batch(BatchArgs b)
{
    constexpr bool WIDTHS = FORM == BATCH_WIDTHS;
    constexpr TbDef d6 = tb_def(k_tb_shapes + 1), d7 = tb_def(k_tb_shapes + 2);
    static_assert(!WIDTHS || (NT == d6.lanes && NT == d7.lanes), "the widths share a launch");
    constexpr int TY6 = d6.rows - 2 * T, TY7 = d7.rows - 2 * T;
    constexpr int F0 = TbGeom<S, TXG, TY, T, NT>::FIELD;
    constexpr int F6 = WIDTHS ? TbGeom<S, d6.txg, WIDTHS ? TY6 : 4, WIDTHS ? T : 1, d6.lanes>::FIELD : 0;
    constexpr int F7 = WIDTHS ? TbGeom<S, d7.txg, WIDTHS ? TY7 : 4, WIDTHS ? T : 1, d7.lanes>::FIELD : 0;
    __shared__ typename Traits<S>::C lds[2 * (F0 > F6 ? (F0 > F7 ? F0 : F7) : (F6 > F7 ? F6 : F7))];
    __shared__ uint4 pre_lds[tb_pre_slots<S, T, NT, NOISE>()];
    const uint32_t r0 = blockIdx.x / (uint32_t)b.slots * (uint32_t)b.slots;
    const uint32_t lb = r0 + xcd_logical_block(blockIdx.x - r0, min((uint32_t)b.slots, gridDim.x - r0));
    const WorkItem w = b.items[lb];
    const SimDesc &d = b.sims[w.sim];
    StepArgs a = b.coef;
    a.nx = d.nx;
    a.ny = d.ny;
    a.nz = d.nz;
    a.zc = d.zc;
    a.F = d.F;
    a.FK = d.FK;
    a.F_f = d.F_f;
    a.FK_f = d.FK_f;
    a.seed = d.seed;
    const S *u = (const S *)d.buf[b.parity][0], *v = (const S *)d.buf[b.parity][1];
    S *un = (S *)d.buf[b.parity ^ 1][0], *vn = (S *)d.buf[b.parity ^ 1][1];
    const uint64_t t0 = NOISE ? (b.t_dev ? *b.t_dev + b.t : b.t) : 0;
    if constexpr (WIDTHS) {
        const int width = item_width(w);
        if (width == 1) return tb_item<S, d6.txg, TY6, T, NT, NOISE>(u, v, un, vn, a, w.bx, w.by, item_bz(w), t0, lds, pre_lds);
        if (width == 2) return tb_item<S, d7.txg, TY7, T, NT, NOISE>(u, v, un, vn, a, w.bx, w.by, item_bz(w), t0, lds, pre_lds);
    }
    tb_item<S, TXG, TY, T, NT, NOISE, FORM != BATCH_PACKED>(u, v, un, vn, a, w.bx, w.by, WIDTHS ? item_bz(w) : w.bz, t0,
                                                             lds, pre_lds);
}

// ------------------------------------------------------------------ launch
// f(shape, T) as constants, where the kernel exists; else `none`.
template <typename S, bool BATCH, int SHAPE, int T, typename R, typename F>
static R with_kernel(int shape, int depth, R none, const F &f)
{
    if constexpr (T > k_tb_depth) {
        return none;
    } else if constexpr (SHAPE > k_tb_shapes + k_tb_narrow) {
        return with_kernel<S, BATCH, 1, T + 1>(shape, depth, none, f);
    } else {
        if (shape != SHAPE || depth != T) return with_kernel<S, BATCH, SHAPE + 1, T>(shape, depth, none, f);
        if constexpr (T <= tb_max_T_shape<S, BATCH>(SHAPE)) return f(Phase<SHAPE>{}, Phase<T>{});
        else return none;
    }
}

template <typename S, int TXG, int TY, int T, int NT>
static hipError_t launch_tb_t(const void *u, const void *v, void *un, void *vn, StepArgs a, hipStream_t st)
{
    a.ntx = (a.nx + TXG * 4 - 1) / (TXG * 4);
    a.nty = (a.ny + TY - 1) / TY;
    const int nzc = (a.nz + a.zc - 1) / a.zc;
    const size_t nb = (size_t)a.ntx * a.nty * nzc;
    if (!grid_fits(nb, NT)) return hipErrorInvalidConfiguration;
    auto go = [&](auto mode) {
        hipLaunchKernelGGL((stencil_tb<S, TXG, TY, T, NT, decltype(mode)::value>), dim3((unsigned)nb), dim3(NT), 0, st,
                           (const S *)u, (const S *)v, (S *)un, (S *)vn, a);
        return hipGetLastError();
    };
    if (a.noise == 0.0) return go(Phase<NOISE_OFF>{});
    if constexpr (tb_noise_64<S, T, NT>()) return go(Phase<NOISE_64>{});
    else if (noise_fits_32(a.nx, a.ny, a.nz)) return go(Phase<NOISE_32>{});
    // (four FP64 buffers of 2^34 cells are 512 GiB: more than the device holds)
    else if constexpr (sizeof(S) == 8) return hipErrorInvalidConfiguration;
    else return go(Phase<NOISE_64>{});
}

template <typename S>
hipError_t dispatch_tb_T(int T, int shape, const void *u, const void *v, void *un, void *vn, const StepArgs &a,
                         hipStream_t st)
{
    return with_kernel<S, false, 1, 1>(shape, T, hipErrorInvalidValue, [&](auto sh, auto depth) {
        constexpr TbDef d = tb_def(decltype(sh)::value);
        constexpr int D = decltype(depth)::value;
        return launch_tb_t<S, d.txg, d.rows - 2 * D, D, d.lanes>(u, v, un, vn, a, st);
    });
}

template <typename S, int TXG, int TY, int T, int NT>
static hipError_t launch_tb_batch_t(const BatchArgs &b, hipStream_t st)
{
    const int grid = b.n_items;
    if (grid < 1 || b.slots < 8) return hipErrorInvalidConfiguration;
    auto go = [&](auto mode) {
        if constexpr (TXG == 16 && NT == 512 && T <= 3) {
            if (b.narrow) {
                hipLaunchKernelGGL((stencil_tb_batch<S, TXG, TY, T, NT, decltype(mode)::value, BATCH_WIDTHS>), dim3(grid), dim3(NT), 0, st, b);
                return hipGetLastError();
            }
        }
        if constexpr (tb_packs<S, T, NT, decltype(mode)::value>()) {
            if (b.n_items > b.slots) {
                hipLaunchKernelGGL((stencil_tb_batch<S, TXG, TY, T, NT, decltype(mode)::value, BATCH_PACKED>), dim3(grid), dim3(NT), 0, st, b);
                return hipGetLastError();
            }
        }
        hipLaunchKernelGGL((stencil_tb_batch<S, TXG, TY, T, NT, decltype(mode)::value, BATCH_PLAIN>), dim3(grid), dim3(NT), 0, st, b);
        return hipGetLastError();
    };
    if (b.coef.noise == 0.0) return go(Phase<NOISE_OFF>{});
    if constexpr (tb_noise_64<S, T, NT>()) return go(Phase<NOISE_64>{});
    else if (b.noise_32) return go(Phase<NOISE_32>{});
    else if constexpr (sizeof(S) == 8) return hipErrorInvalidConfiguration;
    else return go(Phase<NOISE_64>{});
}

template <typename S>
hipError_t batch_T(int T, int shape, const BatchArgs &b, hipStream_t st)
{
    return with_kernel<S, true, 1, 1>(shape, T, hipErrorInvalidValue, [&](auto sh, auto depth) {
        constexpr TbDef d = tb_def(decltype(sh)::value);
        constexpr int D = decltype(depth)::value;
        return launch_tb_batch_t<S, d.txg, d.rows - 2 * D, D, d.lanes>(b, st);
    });
}

template <typename S, int TXG, int TY, int T, int NT>
static int occ_t()
{
    int n = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, stencil_tb_batch<S, TXG, TY, T, NT, NOISE_OFF, BATCH_PLAIN>, NT, 0) != hipSuccess)
        return 1;
    return n > 0 ? n : 1;
}

template <typename S>
int occ_T(int T, int shape)
{
    return with_kernel<S, true, 1, 1>(shape, T, 1, [&](auto sh, auto depth) {
        constexpr TbDef d = tb_def(decltype(sh)::value);
        constexpr int D = decltype(depth)::value;
        return occ_t<S, d.txg, d.rows - 2 * D, D, d.lanes>();
    });
}

template <typename S, int TXG, int TY, int T, int NT>
static int occ_single_t(bool noise)
{
    int n = 0;
    const hipError_t e = noise
                             ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, stencil_tb<S, TXG, TY, T, NT, tb_noise_64<S, T, NT>() ? NOISE_64 : NOISE_32>, NT, 0)
                             : hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, stencil_tb<S, TXG, TY, T, NT, NOISE_OFF>, NT, 0);
    return e == hipSuccess && n > 0 ? n : 0;
}

template <typename S>
int occ_single_T(int T, int shape, bool noise)
{
    return with_kernel<S, false, 1, 1>(shape, T, 0, [&](auto sh, auto depth) {
        constexpr TbDef d = tb_def(decltype(sh)::value);
        constexpr int D = decltype(depth)::value;
        return occ_single_t<S, d.txg, d.rows - 2 * D, D, d.lanes>(noise);
    });
}

// The kernels of a storage type are instantiated in an object of their own
// (GS_TB_STORAGE, set by the build), which the compiler can build side by
// side; the object of storage 0 also holds the functions below.
#define GS_TB_TYPE(X, S, BATCHED)                                                                                          \
    X template hipError_t dispatch_tb_T<S>(int, int, const void *, const void *, void *, void *, const StepArgs &,       \
                                           hipStream_t);                                                                 \
    X template int occ_single_T<S>(int, int, bool);                                                                      \
    BATCHED(X, S)
#define GS_TB_BATCH(X, S)                                                                                                \
    X template hipError_t batch_T<S>(int, int, const BatchArgs &, hipStream_t);                                     \
    X template int occ_T<S>(int, int);
#define GS_TB_SINGLE(X, S)
#if GS_TB_STORAGE == 1
GS_TB_TYPE(, float, GS_TB_BATCH)
#elif GS_TB_STORAGE == 2
GS_TB_TYPE(, bf16, GS_TB_BATCH)
#elif GS_TB_STORAGE == 3
GS_TB_TYPE(, f16, GS_TB_BATCH)
#elif GS_TB_STORAGE == 4
GS_TB_TYPE(, bf16c, GS_TB_SINGLE)
#else
GS_TB_TYPE(extern, float, GS_TB_BATCH)
GS_TB_TYPE(extern, bf16, GS_TB_BATCH)
GS_TB_TYPE(extern, f16, GS_TB_BATCH)
GS_TB_TYPE(extern, bf16c, GS_TB_SINGLE)

int num_tb_shapes() { return k_tb_shapes; }
int num_tb_narrow() { return k_tb_narrow; }

TileShape tb_shape(int shape, int T)
{
    if (shape < 1 || shape > k_tb_shapes + k_tb_narrow) return TileShape{0, 0};
    return TileShape{4 * tb_def(shape).txg, tb_def(shape).rows - 2 * T};
}

template <bool BATCH> static int max_T_for(int shape, int storage)
{
    if (shape < 1 || shape > num_tb_shapes() + (BATCH ? 0 : num_tb_narrow())) return 0;
    switch (storage) {
    case 0: return tb_max_T_shape<double, BATCH>(shape);
    case 1: return tb_max_T_shape<float, BATCH>(shape);
    case 2: return tb_max_T_shape<bf16, BATCH>(shape);
    case 3: return tb_max_T_shape<f16, BATCH>(shape);
    case 4: return BATCH ? 0 : tb_max_T_shape<bf16c, false>(shape);
    }
    return 0;
}

int tb_max_T(int shape, int storage) { return max_T_for<false>(shape, storage); }
int tb_batch_max_T(int shape, int storage) { return max_T_for<true>(shape, storage); }

hipError_t launch_tblock_batch(int storage, int T, int shape, const BatchArgs &b, hipStream_t st)
{
    switch (storage) {
    case 0: return batch_T<double>(T, shape, b, st);
    case 1: return batch_T<float>(T, shape, b, st);
    case 2: return batch_T<bf16>(T, shape, b, st);
    case 3: return batch_T<f16>(T, shape, b, st);
    }
    return hipErrorInvalidValue;
}

int tb_occupancy(int storage, int T, int shape, bool noise)
{
    switch (storage) {
    case 0: return occ_single_T<double>(T, shape, noise);
    case 1: return occ_single_T<float>(T, shape, noise);
    case 2: return occ_single_T<bf16>(T, shape, noise);
    case 3: return occ_single_T<f16>(T, shape, noise);
    case 4: return occ_single_T<bf16c>(T, shape, noise);
    }
    return 0;
}

int tb_batch_occupancy(int storage, int T, int shape)
{
    switch (storage) {
    case 0: return occ_T<double>(T, shape);
    case 1: return occ_T<float>(T, shape);
    case 2: return occ_T<bf16>(T, shape);
    case 3: return occ_T<f16>(T, shape);
    }
    return 1;
}

hipError_t launch_tblock(int storage, int T, int shape, const void *u, const void *v, void *un, void *vn,
                         const StepArgs &a, hipStream_t st)
{
    switch (storage) {
    case 0: return dispatch_tb_T<double>(T, shape, u, v, un, vn, a, st);
    case 1: return dispatch_tb_T<float>(T, shape, u, v, un, vn, a, st);
    case 2: return dispatch_tb_T<bf16>(T, shape, u, v, un, vn, a, st);
    case 3: return dispatch_tb_T<f16>(T, shape, u, v, un, vn, a, st);
    case 4: return dispatch_tb_T<bf16c>(T, shape, u, v, un, vn, a, st);
    }
    return hipErrorInvalidValue;
}

#endif

} // namespace gs
