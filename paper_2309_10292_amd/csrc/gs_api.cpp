// C ABI of libgs (declared in include/gs.h): validation, handle state,
// ping-pong parity, host <-> device conversion, launch selection.
#include "../../include/gs.h"
#include "gs_launch.hpp"
#include "gs_internal.hpp"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <string>
#include <vector>

namespace gsapi {

thread_local std::string g_err;

gs_status fail(gs_status s, const char *fmt, ...) __attribute__((format(printf, 2, 3)));
gs_status fail(gs_status s, const char *fmt, ...)
{
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_err = buf;
    return s;
}

gs_status hip_fail(hipError_t e, const char *what)
{
    return fail(GS_ERR_HIP, "%s: %s (%d)", what, hipGetErrorString(e), (int)e);
}

const uint32_t k_magic = 0x47534d49u; // "GSMI"

size_t storage_bytes(int32_t s)
{
    switch (s) {
    case GS_F64: return 8;
    case GS_F32: return 4;
    case GS_BF16: return 2;
    case GS_F16: return 2;
    case GS_BF16C: return 2;
    }
    return 0;
}

bool aligned(const void *p, size_t a) { return ((uintptr_t)p % a) == 0; }

int device_cus()
{
    int cus = 0, dev = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
        (void)hipGetLastError();
    return cus > 0 ? cus : 256;
}

// Tile indices: 1..num_tiles() select the single-step z-streaming kernel's
// shapes; the next num_tb_shapes() indices select the temporally blocked
// kernel's shapes (any tblock), the next num_blk_shapes() the block
// kernel's (any tblock; z-chunks do not apply to them), and the last
// num_tb_narrow() the temporally blocked kernel's narrow shapes.
int first_blk() { return gs::num_tiles() + gs::num_tb_shapes(); } // block shape s is tile first_blk() + s
int last_blk() { return first_blk() + gs::num_blk_shapes(); }
int total_tiles() { return last_blk() + gs::num_tb_narrow(); }
bool is_blk_tile(int tile) { return tile > first_blk() && tile <= last_blk(); }
bool is_tb_tile(int tile) { return tile > gs::num_tiles() && !is_blk_tile(tile); }
int tb_shape_of(int tile) { return tile <= first_blk() ? tile - gs::num_tiles() : tile - last_blk() + gs::num_tb_shapes(); }
int tb_tile_of(int shape) { return shape <= gs::num_tb_shapes() ? gs::num_tiles() + shape : last_blk() + shape - gs::num_tb_shapes(); }
int tile_max_tblock(int tile, int storage)
{
    if (is_blk_tile(tile)) return GS_MAX_TBLOCK;
    return is_tb_tile(tile) ? gs::tb_max_T(tb_shape_of(tile), storage) : 1;
}

gs_status validate(const gs_params *p)
{
    if (!p) return fail(GS_ERR_INVALID_ARG, "params is NULL");
    if (storage_bytes(p->storage) == 0) return fail(GS_ERR_INVALID_ARG, "unknown storage type %d", p->storage);
    if (p->nx < 4 || p->ny < 4 || p->nz < 4)
        return fail(GS_ERR_UNSUPPORTED, "grid %dx%dx%d: every dimension must be >= 4", p->nx, p->ny, p->nz);
    if (p->nx % 8 != 0) return fail(GS_ERR_UNSUPPORTED, "nx = %d must be a multiple of 8", p->nx);
    const double n = (double)p->nx * p->ny * p->nz;
    if (n * 16.0 > 9.0e18) return fail(GS_ERR_UNSUPPORTED, "grid too large");
    const double c[6] = {p->Du, p->Dv, p->F, p->k, p->dt, p->noise};
    const char *nm[6] = {"Du", "Dv", "F", "k", "dt", "noise"};
    for (int i = 0; i < 6; ++i)
        if (!std::isfinite(c[i])) return fail(GS_ERR_INVALID_ARG, "%s is not finite", nm[i]);
    if (p->Du < 0 || p->Dv < 0) return fail(GS_ERR_INVALID_ARG, "diffusion rates must be >= 0");
    if (p->noise < 0) return fail(GS_ERR_INVALID_ARG, "noise must be >= 0");
    // The FP64 kernels scale the noise by 2^-32 exactly; below this bound the
    // scaled value would be subnormal.
    if (p->noise != 0 && p->noise < 0x1p-990)
        return fail(GS_ERR_UNSUPPORTED, "noise %g below 2^-990 is not supported", p->noise);
    if (p->init_mode != GS_INIT_NONE && p->init_mode != GS_INIT_CUBE)
        return fail(GS_ERR_INVALID_ARG, "unknown init_mode %d", p->init_mode);
    if (p->init_mode == GS_INIT_CUBE) {
        int mn = p->nx < p->ny ? p->nx : p->ny;
        mn = mn < p->nz ? mn : p->nz;
        if (p->cube_side < 1 || p->cube_side > mn)
            return fail(GS_ERR_INVALID_ARG, "cube_side %d outside [1, %d]", p->cube_side, mn);
        if (!std::isfinite(p->cube_u) || !std::isfinite(p->cube_v))
            return fail(GS_ERR_INVALID_ARG, "cube values must be finite");
    }
    if (p->tblock < 0 || p->tblock > GS_MAX_TBLOCK)
        return fail(GS_ERR_INVALID_ARG, "tblock %d outside [0, %d]", p->tblock, GS_MAX_TBLOCK);
    if (p->tile < 0 || p->tile > total_tiles())
        return fail(GS_ERR_INVALID_ARG, "tile %d outside [0, %d]", p->tile, total_tiles());
    if (p->tile >= 1 && p->tile <= gs::num_tiles() && p->tblock > 1)
        return fail(GS_ERR_INVALID_ARG, "tile %d is a single-step tile; tblock must be 0 or 1", p->tile);
    if (p->tile >= 1 && p->tblock > tile_max_tblock(p->tile, p->storage))
        return fail(GS_ERR_INVALID_ARG, "tile %d fuses at most %d steps for this storage type", p->tile,
                    tile_max_tblock(p->tile, p->storage));
    if (p->zchunk < 0) return fail(GS_ERR_INVALID_ARG, "zchunk %d < 0", p->zchunk);
    if (p->reserved != 0) return fail(GS_ERR_INVALID_ARG, "reserved field must be 0");
    return GS_OK;
}

// Host rounding used by gs_write: FP64 -> FP32 (nearest-even, the C cast),
// then FP32 -> 16-bit nearest-even.
uint16_t host_bf16(float f)
{
    uint32_t u;
    std::memcpy(&u, &f, 4);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40u);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}
gs_status write_field(void *dev, int32_t storage, size_t n, const double *host, hipStream_t st, int field)
{
    const size_t es = storage_bytes(storage);
    std::vector<unsigned char> stage;
    const void *src = host;
    if (storage != GS_F64) {
        stage.resize(n * es);
        if (storage == GS_F32) {
            float *d = (float *)stage.data();
            for (size_t i = 0; i < n; ++i) d[i] = (float)host[i];
        } else if (storage == GS_BF16) {
            uint16_t *d = (uint16_t *)stage.data();
            for (size_t i = 0; i < n; ++i) d[i] = host_bf16((float)host[i]);
        } else if (storage == GS_BF16C) {
            // u: 1 - u formed in FP64, then rounded to FP32 and to BF16
            uint16_t *d = (uint16_t *)stage.data();
            if (field == 0)
                for (size_t i = 0; i < n; ++i) d[i] = host_bf16((float)(1.0 - host[i]));
            else
                for (size_t i = 0; i < n; ++i) d[i] = host_bf16((float)host[i]);
        } else {
            _Float16 *d = (_Float16 *)stage.data();
            for (size_t i = 0; i < n; ++i) d[i] = (_Float16)(float)host[i];
        }
        src = stage.data();
    }
    hipError_t e = hipMemcpyAsync(dev, src, n * es, hipMemcpyHostToDevice, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    return e == hipSuccess ? GS_OK : hip_fail(e, "host-to-device copy");
}

gs_status diagnostics(int32_t storage, const void *u, const void *v, size_t n, void *ws, hipStream_t st,
                      gs_diag *out)
{
    hipError_t e = gs::launch_diagnostics(storage, u, v, n, ws, st);
    if (e != hipSuccess) return hip_fail(e, "diagnostics launch");
    double r[9];
    e = hipMemcpyAsync(r, (char *)ws + gs::diag_result_offset(), sizeof r, hipMemcpyDeviceToHost, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    if (e != hipSuccess) return hip_fail(e, "diagnostics copy");
    out->sum_u = r[0] + r[1];
    out->sum_v = r[2] + r[3];
    out->min_u = r[4];
    out->max_u = r[5];
    out->min_v = r[6];
    out->max_v = r[7];
    out->nonfinite = (int64_t)r[8];
    if (out->nonfinite > 0) return fail(GS_ERR_NONFINITE, "%lld non-finite values", (long long)out->nonfinite);
    return GS_OK;
}

size_t counter_offset() { return (gs::diag_workspace_bytes() + 255) / 256 * 256; }

} // namespace gsapi

using namespace gsapi;

struct GraphCache {
    hipGraphExec_t exec = nullptr;
    int64_t n = -1;
    int parity = -1;
    int tile = 0, tblock = 0, zc = 0;
};

struct gs_sim {
    uint32_t magic;
    gs_params p;
    void *buf[2][2]; // [parity][field]
    int parity;      // buffers holding the current state
    uint64_t step;   // global step index of the current state
    void *ws;
    hipStream_t stream;
    int tile;
    int zc;
    int tblock;
    size_t n;
    GraphCache graph;
    hipStream_t capture_stream;
    ReadStage reads;
};

namespace {

gs_status check(gs_sim *s)
{
    if (!s || s->magic != k_magic) return fail(GS_ERR_STATE, "invalid or destroyed handle");
    return GS_OK;
}

// Library choice of the launch configuration before any tuning (from the
// MI355X autotuner sweeps at 64^3 .. 1024^3, with and without noise): the
// temporally blocked kernel above the smallest sizes. Large grids (>= 64 M cells): FP64
// fuses three steps in the 512-lane 64 x 22 tile; with noise the other
// storage types fuse two steps in the same tile (the Philox blocks of deeper
// fusion cost more than the traffic they save); without noise the 16-bit types
// fuse two steps in the 512-lane tile and FP32 three in the 1024-lane one,
// where two are bound by HBM (1024^3: 1.60 ms per step against 1.88; 640^3 0.44
// against 0.50), unless its tiles of 50 rows cover the grid worse than those of
// two steps (512^3: 0.24 against 0.22).
// Smaller grids take the launch that default_stream estimates fastest (where
// gs_params sets a part of it, two steps in 256-lane workgroups below 4 M cells
// and above that in the 768-lane tile for FP64 and the 512-lane one for the
// others). The single-step kernel (tiles 1..4) runs when asked for. The smallest
// and the narrowest grids take the block kernel (default_block), unless gs_params
// sets the z-chunk.
double grid_cells(const gs_params &p) { return (double)p.nx * p.ny * p.nz; }
bool large_grid(const gs_params &p) { return grid_cells(p) >= 64.0 * 1024 * 1024; }

// Block kernel of small grids: shape (0: not taken) and steps per launch.
// A z-streaming workgroup is a serial chain of planes, two barriers each: on a
// grid that does not fill the chip a launch takes 8 to 10 us whatever its size.
// A block is loaded at once, so while there are blocks for about every CU a
// launch costs its latency and more fused steps pay (us per step, FP64 without
// noise, z-streaming against the block kernel): 32^3 4.53 -> 1.72 (8x4x4, four
// steps; with noise, whose Philox blocks add up, 2.16 against 2.09 with three;
// 40^3, two blocks per CU: 2.40 with four, 2.23 with three), 48^3 4.77 -> 2.41
// (16x8x4, three), 64^3 4.89 -> 3.18 (16x8x8, three). With more blocks than that
// their halos decide: 72^3 7.17 -> 4.73 and 80^3 6.49 -> 4.97 (16x8x4, two
// steps), while 88^3 ties and 128 x 106 x 75 loses 15 %. The z-streaming tile is
// 64 x 10 cells, so what it wastes on narrow rows counts too: 16 x 250 x 250
// 18.6 -> 7.9 and 16 x 600 x 600 72 -> 31 (16x8x8, one step); 32 x 150 x 200 gains
// 6 % in FP64 and loses 5 % in BF16 with noise, 24 x 640 x 640 loses 20 %. The numbers
// of blocks are per CU of the 256 that this was measured with.
struct BlockChoice {
    int shape, T;
};
BlockChoice default_block(const gs_params &p, int cus)
{
    if (p.zchunk) return BlockChoice{0, 0}; // the caller's z-chunk has no meaning for blocks
    auto up = [](int n, int t) { return (double)((n + t - 1) / t); };
    auto blocks = [&](int shape) {
        const gs::BlkShape b = gs::blk_shape(shape);
        return up(p.nx, b.bx) * up(p.ny, b.by) * up(p.nz, b.bz);
    };
    if (blocks(1) <= 2 * cus) return BlockChoice{1, 16 * blocks(1) <= 25 * cus ? 4 : 3};
    if (blocks(2) <= cus) return BlockChoice{2, 3};
    if (blocks(3) <= cus) return BlockChoice{3, 3};
    const double streamed = 64 * up(p.nx, 64) * 10 * up(p.ny, 10) * p.nz; // cells its tiles cover
    if (grid_cells(p) < 4.0 * 1024 * 1024)
        return 32 * blocks(2) <= 75 * cus || 512 * blocks(2) <= (grid_cells(p) < 600e3 ? 0.63 : 0.45) * streamed ? BlockChoice{2, 2}
                                                                                                      : BlockChoice{0, 0};
    return !large_grid(p) && 1024 * blocks(3) <= 0.3 * streamed ? BlockChoice{3, 1} : BlockChoice{0, 0};
}

int default_tile(const gs_params &p, int cus)
{
    const BlockChoice b = default_block(p, cus);
    if (b.shape) return first_blk() + b.shape;
    const int tb = gs::num_tiles(); // tiles tb + 1 .. tb + 5 are the blocked shapes 1..5
    if (grid_cells(p) < 4.0 * 1024 * 1024) return tb + 1;
    int tile = tb + 2;
    if (!large_grid(p) && p.storage == GS_F64) tile = tb + 4;
    if (large_grid(p) && p.storage == GS_F32 && p.noise == 0.0) tile = tb + 5;
    // a caller's tblock may be more than the larger tiles fuse; the 512-lane one fuses any
    return p.tblock <= tile_max_tblock(tile, p.storage) ? tile : tb + 2;
}

int default_tblock(const gs_params &p, int tile, int cus)
{
    if (tile <= gs::num_tiles()) return 1;
    const BlockChoice b = default_block(p, cus);
    if (is_blk_tile(tile)) return tile == first_blk() + b.shape ? b.T : 2;
    int T = 2;
    if (large_grid(p) && p.storage == GS_F64) T = 3;
    if (large_grid(p) && p.storage == GS_F32 && tile == gs::num_tiles() + 5) {
        auto rows = [&](int depth) {
            const int ty = gs::tb_shape(5, depth).ty;
            return (double)((p.ny + ty - 1) / ty * ty);
        };
        if (rows(3) <= 1.05 * rows(2)) T = 3;
    }
    const int mt = tile_max_tblock(tile, p.storage);
    return T < mt ? T : mt;
}

// z-chunks the autotuner sweeps.
const int k_zchunks[] = {4, 8, 16, 32, 64, 128, 256, 512};

// Default z-chunk: a workgroup of a chunk of zc output planes streams
// zc + 2T planes, and nb workgroups on `slots` resident places (CUs times
// workgroups per CU) take ceil(nb / slots) rounds, so the sweep costs about
// ceil(nb / slots) (zc + 2T) plane times; the partly filled last round costs
// up to a fifth of the throughput at 512^3 with a fixed chunk. Chunks that
// leave fewer than three rounds are slower than this predicts on large grids
// (every CU then starts and drains its workgroups at once), so the cheapest
// chunk with at least three rounds (two below 64 M cells, where longer
// chunks measured faster) is taken (the larger one on ties), else the
// shortest chunk. The single-step kernel keeps chunks of at most 32 planes (longer
// ones measured slower at 1024^3 although the estimate favours them).
// Without the occupancy figures it falls back to fixed chunks.
int default_zc(const gs_params &p, int tile, int tblock)
{
    if (is_blk_tile(tile)) return std::min(gs::blk_shape(tile - first_blk()).bz, p.nz);
    int cus = 0, dev = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
        cus = 0;
    const bool tb = is_tb_tile(tile);
    const int occ = tb ? gs::tb_occupancy(p.storage, tblock, tb_shape_of(tile), p.noise != 0.0)
                       : gs::step_occupancy(p.storage, tile, p.noise != 0.0);
    const gs::TileShape t = tb ? gs::tb_shape(tb_shape_of(tile), tblock) : gs::tile_shape(tile, p.storage);
    if (cus > 0 && occ > 0 && t.tx > 0 && t.ty > 0) {
        const double slots = (double)cus * occ;
        const double tiles = (double)((p.nx + t.tx - 1) / t.tx) * (double)((p.ny + t.ty - 1) / t.ty);
        const int T = tb ? tblock : 1;
        const double min_rounds = large_grid(p) ? 3.0 : 2.0;
        double best = 1e300;
        int bz = 0;
        for (int z : k_zchunks) {
            const int zc = z < p.nz ? z : p.nz;
            const double nb = tiles * (double)((p.nz + zc - 1) / zc);
            if (nb < min_rounds * slots || (!tb && z > 32)) continue;
            const double cost = std::ceil(nb / slots) * (double)(zc + 2 * T);
            if (cost <= best) {
                best = cost;
                bz = zc;
            }
        }
        if (bz == 0) bz = k_zchunks[0] < p.nz ? k_zchunks[0] : p.nz;
        return bz;
    }
    int z = 16;
    if (large_grid(p))
        z = tile <= gs::num_tiles() ? 32 : p.storage == GS_F64 ? 128 : p.storage == GS_F32 ? 32 : 64;
    return p.nz < z ? p.nz : z;
}

// Launch of grids between the block kernel's and 64 M cells when gs_params leaves
// all of it to the library: the blocked shape, depth and z-chunk of least
// estimated time per step. A launch of nb workgroups on CUs that hold occ each
// runs nb / (CUs occ) full rounds and a part of one; a round takes
// (zc + 2T - 1) plane times (the chunk, the planes its levels run ahead and one
// for its start), and a plane of a CU with n workgroups fixed + n each, in us.
// The constants are least-squares fits over 25 grids of 0.4 to 57 M cells and 14
// chunks each (10 % standard deviation); over those grids, six storage and noise
// cases, the choice takes 0.9 % longer than the best measured launch and is
// 15 % faster than fixed shapes with power-of-two chunks: FP64 192^3 39.8 ->
// 27.7 us per step, 320^3 143 -> 103, 128^3 14.6 -> 12.5, FP32 256^3 39.1 -> 34.6,
// BF16 320 x 100 x 200 15.6 -> 11.9.
// The narrow shapes cost what shape 2 does, and up to a fifth more where the tiles are
// as many (448 x 159 x 300 BF16 28.6 against 33.8, 184 x 250 x 100 FP64 19.2 against
// 22.4): they have to look 10% faster. Over 42 grids, six cases each, 60 launches
// change and take 0.85 of their time: 24 x 640 x 640 FP64 75.3 -> 40.7 and BF16 32.4 ->
// 18.9, 72 x 300 x 300 FP32 22.4 -> 18.7, 272^3 FP64 84.0 -> 75.4; at worst 184 x
// 250 x 100 FP64 with noise 21.8 -> 23.2.
struct StreamCost {
    int shape, T, occ;
    double fixed[2], each[2]; // without and with noise
};
struct StreamChoice {
    int shape, T, zc;
};
StreamChoice default_stream(const gs_params &p, int cus)
{
    static const StreamCost f64[] = {{1, 2, 2, {0.70, 0.84}, {0.55, 0.57}},
                                     {2, 2, 1, {0.96, 1.10}, {0.96, 1.10}},
                                     {2, 3, 1, {1.22, 1.51}, {1.23, 1.51}},
                                     {6, 2, 1, {0.96, 1.10}, {0.96, 1.10}},
                                     {6, 3, 1, {1.22, 1.51}, {1.23, 1.51}},
                                     {7, 2, 1, {0.96, 1.10}, {0.96, 1.10}},
                                     {7, 3, 1, {1.22, 1.51}, {1.23, 1.51}}};
    static const StreamCost f32[] = {{1, 2, 4, {0.75, 0.90}, {0.29, 0.33}},
                                     {2, 2, 2, {0.89, 1.11}, {0.59, 0.65}},
                                     {5, 2, 1, {1.16, 1.40}, {1.16, 1.40}},
                                     {6, 2, 2, {0.89, 1.11}, {0.59, 0.65}},
                                     {7, 2, 2, {0.89, 1.11}, {0.59, 0.65}}};
    static const StreamCost b16[] = {{1, 2, 4, {0.68, 0.84}, {0.17, 0.19}},
                                     {2, 2, 2, {0.73, 0.99}, {0.38, 0.39}},
                                     {5, 2, 1, {0.84, 1.05}, {0.84, 1.05}},
                                     {6, 2, 2, {0.73, 0.99}, {0.38, 0.39}},
                                     {7, 2, 2, {0.73, 0.99}, {0.38, 0.39}}};
    const StreamCost *table = p.storage == GS_F64 ? f64 : p.storage == GS_F32 ? f32 : b16;
    const int noise = p.noise != 0.0;
    StreamChoice best = {1, 2, 4};
    double best_us = 1e300;
    for (int i = 0; i < (p.storage == GS_F64 ? 7 : 5); ++i) {
        const StreamCost &c = table[i];
        const gs::TileShape t = gs::tb_shape(c.shape, c.T);
        const int64_t tiles = (int64_t)((p.nx + t.tx - 1) / t.tx) * ((p.ny + t.ty - 1) / t.ty);
        for (int z = 3; z <= 64 && z <= p.nz; ++z) {
            const int64_t nb = tiles * ((p.nz + z - 1) / z), full = nb / (cus * c.occ), rest = nb % (cus * c.occ);
            double plane = full * (c.fixed[noise] + c.occ * c.each[noise]);
            if (rest) plane += c.fixed[noise] + (double)((rest + cus - 1) / cus) * c.each[noise];
            double us = (2.5 + (z + 2 * c.T - 1) * plane) / c.T; // 2.5: a launch
            if (c.shape > gs::num_tb_shapes()) us *= 1.1;
            if (us <= best_us) {
                best_us = us;
                best = StreamChoice{c.shape, c.T, z};
            }
        }
    }
    return best;
}

gs::StepArgs make_args(const gs_sim *s)
{
    gs::StepArgs a = {};
    a.nx = s->p.nx;
    a.ny = s->p.ny;
    a.nz = s->p.nz;
    a.zc = s->zc;
    a.Du = s->p.Du;
    a.Dv = s->p.Dv;
    a.F = s->p.F;
    a.FK = s->p.F + s->p.k;
    a.dt = s->p.dt;
    a.noise = s->p.noise;
    a.noise_s = std::ldexp(a.noise, -31);
    a.noise_h = std::ldexp(a.noise, -32);
    a.Du6_f = (float)(a.Du / 6.0);
    a.Dv6_f = (float)(a.Dv / 6.0);
    a.F_f = (float)a.F;
    a.FK_f = (float)a.FK;
    a.dt_f = (float)a.dt;
    a.noise_s_f = (float)a.noise_s;
    a.noise_h_f = (float)a.noise_h;
    a.seed = s->p.seed;
    a.t = s->step;
    a.t_dev = nullptr;
    return a;
}

// Enqueues n steps starting from buffer pair *parity on stream st; with
// t_dev set, kernels read the base step index from device memory and take
// their offset from it. Leaves the final parity in *parity.
hipError_t enqueue_steps(gs_sim *s, int64_t n, hipStream_t st, const uint64_t *t_dev, int *parity)
{
    int64_t left = n, off = 0;
    while (left > 0) {
        gs::StepArgs a = make_args(s);
        if (t_dev) {
            a.t = (uint64_t)off;
            a.t_dev = t_dev;
        } else {
            a.t = s->step + (uint64_t)off;
        }
        const int q = *parity;
        hipError_t e;
        int done = 1;
        if (is_blk_tile(s->tile)) {
            done = gs::next_depth(left, s->tblock);
            e = gs::launch_block(s->p.storage, done, s->tile - first_blk(), s->buf[q][0], s->buf[q][1],
                                 s->buf[q ^ 1][0], s->buf[q ^ 1][1], a, st);
        } else if (is_tb_tile(s->tile)) {
            done = gs::next_depth(left, s->tblock);
            e = gs::launch_tblock(s->p.storage, done, tb_shape_of(s->tile), s->buf[q][0], s->buf[q][1],
                                  s->buf[q ^ 1][0], s->buf[q ^ 1][1], a, st);
        } else {
            e = gs::launch_step(s->p.storage, s->tile, s->buf[q][0], s->buf[q][1], s->buf[q ^ 1][0],
                                s->buf[q ^ 1][1], a, st);
        }
        if (e != hipSuccess) return e;
        *parity ^= 1;
        left -= done;
        off += done;
    }
    return hipSuccess;
}

void drop_graph(gs_sim *s)
{
    if (s->graph.exec) (void)hipGraphExecDestroy(s->graph.exec);
    s->graph = GraphCache();
}

} // namespace

extern "C" {

const char *gs_version(void) { return "gs-mi355x 0.1 (gfx950)"; }

const char *gs_last_error(void) { return g_err.c_str(); }

// Workspace layout: diagnostic partials, then (256-byte aligned) the step
// counter read by graph replays.
size_t gs_workspace_bytes(const gs_params *p)
{
    if (validate(p) != GS_OK) return 0;
    return counter_offset() + 256;
}

int32_t gs_num_tiles(void) { return total_tiles(); }

gs_status gs_tile_info(int32_t tile, int32_t storage, int32_t tblock, int32_t *tx, int32_t *ty, int32_t *max_tblock)
{
    if (tile < 1 || tile > total_tiles()) return fail(GS_ERR_INVALID_ARG, "tile %d out of range", tile);
    if (storage_bytes(storage) == 0) return fail(GS_ERR_INVALID_ARG, "unknown storage type %d", storage);
    const int mt = tile_max_tblock(tile, storage);
    if (tblock < 1 || tblock > mt) return fail(GS_ERR_INVALID_ARG, "tblock %d outside [1, %d] for tile %d", tblock, mt, tile);
    gs::TileShape t;
    if (is_blk_tile(tile)) {
        const gs::BlkShape b = gs::blk_shape(tile - first_blk());
        t = gs::TileShape{b.bx, b.by};
    } else {
        t = is_tb_tile(tile) ? gs::tb_shape(tb_shape_of(tile), tblock) : gs::tile_shape(tile, storage);
    }
    if (tx) *tx = t.tx;
    if (ty) *ty = t.ty;
    if (max_tblock) *max_tblock = mt;
    return GS_OK;
}

gs_status gs_init(const gs_params *p, void *u0, void *v0, void *u1, void *v1, void *workspace,
                  void *hip_stream, gs_sim **out)
{
    if (!out) return fail(GS_ERR_INVALID_ARG, "out is NULL");
    *out = nullptr;
    gs_status st = validate(p);
    if (st != GS_OK) return st;
    void *b[4] = {u0, v0, u1, v1};
    const char *nm[4] = {"u0", "v0", "u1", "v1"};
    for (int i = 0; i < 4; ++i) {
        if (!b[i]) return fail(GS_ERR_INVALID_ARG, "%s is NULL", nm[i]);
        if (!aligned(b[i], 256)) return fail(GS_ERR_INVALID_ARG, "%s is not 256-byte aligned", nm[i]);
        for (int j = 0; j < i; ++j)
            if (b[i] == b[j]) return fail(GS_ERR_INVALID_ARG, "%s aliases %s", nm[i], nm[j]);
    }
    if (!workspace) return fail(GS_ERR_INVALID_ARG, "workspace is NULL");
    if (!aligned(workspace, 256)) return fail(GS_ERR_INVALID_ARG, "workspace is not 256-byte aligned");

    gs_sim *s = new (std::nothrow) gs_sim();
    if (!s) return fail(GS_ERR_INVALID_ARG, "out of host memory");
    s->magic = k_magic;
    s->p = *p;
    s->buf[0][0] = u0;
    s->buf[0][1] = v0;
    s->buf[1][0] = u1;
    s->buf[1][1] = v1;
    s->parity = 0;
    s->step = p->step0;
    s->ws = workspace;
    s->stream = (hipStream_t)hip_stream;
    const int cus = device_cus();
    s->tile = p->tile ? p->tile : default_tile(*p, cus);
    s->tblock = p->tblock ? p->tblock : default_tblock(*p, s->tile, cus);
    s->zc = p->zchunk ? (p->zchunk < p->nz ? p->zchunk : p->nz) : default_zc(*p, s->tile, s->tblock);
    if (p->tile == 0 && p->tblock == 0 && p->zchunk == 0) {
        if (!large_grid(*p) && !default_block(*p, cus).shape) {
            const StreamChoice c = default_stream(*p, cus);
            s->tile = tb_tile_of(c.shape);
            s->tblock = c.T;
            s->zc = c.zc;
        }
        // a configuration recorded by gs_tune for this grid class, if any
        TuneVal v;
        const TuneKey key = {TUNE_SINGLE, p->storage, p->nx, p->ny, p->nz, p->noise != 0.0};
        if (tune_cache_lookup(key, &v) && v.tile >= 1 && v.tile <= total_tiles() && v.tblock >= 1 &&
            v.tblock <= tile_max_tblock(v.tile, p->storage) && v.zchunk >= 1) {
            s->tile = v.tile;
            s->tblock = v.tblock;
            s->zc = v.zchunk < p->nz ? v.zchunk : p->nz;
        }
    }
    s->n = (size_t)p->nx * p->ny * p->nz;
    s->graph = GraphCache();
    s->capture_stream = nullptr;

    if (p->init_mode == GS_INIT_CUBE) {
        hipError_t e = gs::launch_init_cube(p->storage, u0, v0, p->nx, p->ny, p->nz, p->cube_side, p->cube_u,
                                            p->cube_v, s->stream);
        if (e != hipSuccess) {
            s->magic = 0;
            delete s;
            return hip_fail(e, "init kernel launch");
        }
    }
    *out = s;
    return GS_OK;
}

gs_status gs_step(gs_sim *s, int64_t n_steps)
{
    gs_status st = check(s);
    if (st != GS_OK) return st;
    if (n_steps < 0) return fail(GS_ERR_INVALID_ARG, "n_steps = %lld < 0", (long long)n_steps);
    int parity = s->parity;
    hipError_t e = enqueue_steps(s, n_steps, s->stream, nullptr, &parity);
    if (e != hipSuccess) return hip_fail(e, "step kernel launch");
    s->parity = parity;
    s->step += (uint64_t)n_steps;
    return GS_OK;
}

gs_status gs_read(gs_sim *s, double *u_host, double *v_host)
{
    gs_status st = check(s);
    if (st != GS_OK) return st;
    double *dst[2] = {u_host, v_host};
    st = read_fields(s->reads, s->buf[s->parity], s->p.storage, s->n, dst, s->stream);
    if (st != GS_OK) return st;
    hipError_t e = hipStreamSynchronize(s->stream);
    if (e != hipSuccess) return hip_fail(e, "gs_read sync");
    return GS_OK;
}

gs_status gs_write(gs_sim *s, const double *u_host, const double *v_host)
{
    gs_status st = check(s);
    if (st != GS_OK) return st;
    const double *srcs[2] = {u_host, v_host};
    hipError_t e = hipStreamSynchronize(s->stream);
    if (e != hipSuccess) return hip_fail(e, "gs_write sync");
    for (int f = 0; f < 2; ++f) {
        if (!srcs[f]) continue;
        st = write_field(s->buf[s->parity][f], s->p.storage, s->n, srcs[f], s->stream, f);
        if (st != GS_OK) return st;
    }
    return GS_OK;
}

gs_status gs_current(gs_sim *s, void **u_dev, void **v_dev, uint64_t *step)
{
    gs_status st = check(s);
    if (st != GS_OK) return st;
    if (u_dev) *u_dev = s->buf[s->parity][0];
    if (v_dev) *v_dev = s->buf[s->parity][1];
    if (step) *step = s->step;
    return GS_OK;
}

gs_status gs_diagnostics(gs_sim *s, gs_diag *out)
{
    gs_status st = check(s);
    if (st != GS_OK) return st;
    if (!out) return fail(GS_ERR_INVALID_ARG, "out is NULL");
    return diagnostics(s->p.storage, s->buf[s->parity][0], s->buf[s->parity][1], s->n, s->ws, s->stream, out);
}

gs_status gs_sync(gs_sim *s)
{
    gs_status st = check(s);
    if (st != GS_OK) return st;
    hipError_t e = hipStreamSynchronize(s->stream);
    if (e != hipSuccess) return hip_fail(e, "gs_sync");
    return GS_OK;
}

gs_status gs_destroy(gs_sim *s)
{
    gs_status st = check(s);
    if (st != GS_OK) return st;
    hipError_t e = hipStreamSynchronize(s->stream);
    drop_graph(s);
    if (s->capture_stream) (void)hipStreamDestroy(s->capture_stream);
    s->magic = 0;
    delete s;
    if (e != hipSuccess) return hip_fail(e, "gs_destroy sync");
    return GS_OK;
}

gs_status gs_set_config(gs_sim *s, int32_t tile, int32_t tblock, int32_t zchunk)
{
    gs_status st = check(s);
    if (st != GS_OK) return st;
    if (tile < 1 || tile > total_tiles()) return fail(GS_ERR_INVALID_ARG, "tile %d out of range", tile);
    const int mt = tile_max_tblock(tile, s->p.storage);
    if (tblock < 1 || tblock > mt) return fail(GS_ERR_INVALID_ARG, "tblock %d outside [1, %d] for tile %d", tblock, mt, tile);
    if (zchunk < 1) return fail(GS_ERR_INVALID_ARG, "zchunk %d < 1", zchunk);
    s->tile = tile;
    s->tblock = tblock;
    s->zc = zchunk < s->p.nz ? zchunk : s->p.nz;
    return GS_OK;
}

gs_status gs_get_config(gs_sim *s, int32_t *tile, int32_t *tblock, int32_t *zchunk)
{
    gs_status st = check(s);
    if (st != GS_OK) return st;
    if (tile) *tile = s->tile;
    if (tblock) *tblock = s->tblock;
    if (zchunk) *zchunk = s->zc;
    return GS_OK;
}

gs_status gs_tune(gs_sim *s, int32_t reps, gs_tune_entry *table, int32_t capacity, int32_t *n_entries)
{
    gs_status st = check(s);
    if (st != GS_OK) return st;
    if (reps < 1) return fail(GS_ERR_INVALID_ARG, "reps %d < 1", reps);
    if (capacity < 0 || (capacity > 0 && !table)) return fail(GS_ERR_INVALID_ARG, "bad table/capacity");
    const int *zcs = k_zchunks;
    hipEvent_t e0 = nullptr, e1 = nullptr;
    hipError_t e = hipEventCreate(&e0);
    if (e == hipSuccess) e = hipEventCreate(&e1);
    if (e != hipSuccess) {
        if (e0) (void)hipEventDestroy(e0);
        return hip_fail(e, "gs_tune events");
    }
    const int save_tile = s->tile, save_tb = s->tblock, save_zc = s->zc;
    double best = 1e300;
    int bt = save_tile, bT = save_tb, bz = save_zc;
    int count = 0;
    for (int tile = 1; tile <= total_tiles() && e == hipSuccess; ++tile) {
        for (int T = 1; T <= tile_max_tblock(tile, s->p.storage) && e == hipSuccess; ++T) {
            int last_zc = -1;
            for (int zi = 0; zi < (int)(sizeof k_zchunks / sizeof k_zchunks[0]) && e == hipSuccess; ++zi) {
                int zc = zcs[zi] < s->p.nz ? zcs[zi] : s->p.nz;
                if (is_blk_tile(tile)) zc = default_zc(s->p, tile, T); // the block's own planes: one candidate
                if (zc == last_zc) continue;
                last_zc = zc;
                s->tile = tile;
                s->tblock = T;
                s->zc = zc;
                // Reads the current pair and writes the other one; the state
                // and the step index are left unchanged.
                int par = s->parity;
                e = enqueue_steps(s, T, s->stream, nullptr, &par); // warm-up
                if (e == hipErrorInvalidConfiguration) { // more workgroups than a launch takes: no candidate
                    e = hipSuccess;
                    continue;
                }
                if (e == hipSuccess) e = hipEventRecord(e0, s->stream);
                for (int r = 0; r < reps && e == hipSuccess; ++r) {
                    par = s->parity;
                    e = enqueue_steps(s, T, s->stream, nullptr, &par);
                }
                if (e == hipSuccess) e = hipEventRecord(e1, s->stream);
                if (e == hipSuccess) e = hipEventSynchronize(e1);
                float ms = 0.f;
                if (e == hipSuccess) e = hipEventElapsedTime(&ms, e0, e1);
                if (e != hipSuccess) break;
                const double per_step = (double)ms / (reps * T);
                if (count < capacity) {
                    table[count].tile = tile;
                    table[count].tblock = T;
                    table[count].zchunk = zc;
                    table[count].reserved = 0;
                    table[count].ms_per_step = per_step;
                }
                ++count;
                if (per_step < best) {
                    best = per_step;
                    bt = tile;
                    bT = T;
                    bz = zc;
                }
            }
        }
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (e != hipSuccess) {
        s->tile = save_tile;
        s->tblock = save_tb;
        s->zc = save_zc;
        return hip_fail(e, "gs_tune");
    }
    s->tile = bt;
    s->tblock = bT;
    s->zc = bz;
    if (n_entries) *n_entries = count;
    const TuneKey key = {TUNE_SINGLE, s->p.storage, s->p.nx, s->p.ny, s->p.nz, s->p.noise != 0.0};
    if (!tune_cache_store(key, TuneVal{bt, bT, bz, best}))
        return fail(GS_ERR_INVALID_ARG, "tuned, but the table %s could not be written", tune_cache_path());
    return GS_OK;
}

gs_status gs_step_graph(gs_sim *s, int64_t n_steps)
{
    gs_status st = check(s);
    if (st != GS_OK) return st;
    if (n_steps < 0) return fail(GS_ERR_INVALID_ARG, "n_steps = %lld < 0", (long long)n_steps);
    if (n_steps == 0) return GS_OK;
    GraphCache &g = s->graph;
    uint64_t *t_dev = (uint64_t *)((char *)s->ws + counter_offset());
    hipError_t e = hipSuccess;
    int end_parity = s->parity;
    if (!(g.exec && g.n == n_steps && g.parity == s->parity && g.tile == s->tile && g.tblock == s->tblock &&
          g.zc == s->zc)) {
        drop_graph(s);
        if (!s->capture_stream) {
            e = hipStreamCreateWithFlags(&s->capture_stream, hipStreamNonBlocking);
            if (e != hipSuccess) return hip_fail(e, "capture stream");
        }
        hipGraph_t graph = nullptr;
        e = hipStreamBeginCapture(s->capture_stream, hipStreamCaptureModeThreadLocal);
        if (e != hipSuccess) return hip_fail(e, "begin capture");
        int par = s->parity;
        hipError_t le = enqueue_steps(s, n_steps, s->capture_stream, t_dev, &par);
        e = hipStreamEndCapture(s->capture_stream, &graph);
        if (le != hipSuccess) {
            if (graph) (void)hipGraphDestroy(graph);
            return hip_fail(le, "capture launches");
        }
        if (e != hipSuccess) return hip_fail(e, "end capture");
        e = hipGraphInstantiate(&g.exec, graph, nullptr, nullptr, 0);
        (void)hipGraphDestroy(graph);
        if (e != hipSuccess) {
            g = GraphCache();
            return hip_fail(e, "graph instantiate");
        }
        g.n = n_steps;
        g.parity = s->parity;
        g.tile = s->tile;
        g.tblock = s->tblock;
        g.zc = s->zc;
    }
    // The captured kernels take their step index from the device counter.
    e = gs::launch_set_u64(t_dev, s->step, s->stream);
    if (e != hipSuccess) return hip_fail(e, "step counter");
    e = hipGraphLaunch(g.exec, s->stream);
    if (e != hipSuccess) return hip_fail(e, "graph launch");
    const int64_t launches = (n_steps + s->tblock - 1) / s->tblock; // tblock is 1 for the single-step tiles
    if (launches & 1) end_parity ^= 1;
    s->parity = end_parity;
    s->step += (uint64_t)n_steps;
    return GS_OK;
}

gs_status gs_set_step(gs_sim *s, uint64_t step)
{
    gs_status st = check(s);
    if (st != GS_OK) return st;
    s->step = step;
    return GS_OK;
}

gs_status gs_fill_cube(gs_sim *s, int32_t x0, int32_t y0, int32_t z0, int32_t side, double cu, double cv)
{
    gs_status st = check(s);
    if (st != GS_OK) return st;
    int mn = s->p.nx < s->p.ny ? s->p.nx : s->p.ny;
    mn = mn < s->p.nz ? mn : s->p.nz;
    if (side < 1 || side > mn) return fail(GS_ERR_INVALID_ARG, "side %d outside [1, %d]", side, mn);
    if (x0 < 0 || y0 < 0 || z0 < 0 || x0 >= s->p.nx || y0 >= s->p.ny || z0 >= s->p.nz)
        return fail(GS_ERR_INVALID_ARG, "corner outside the grid");
    if (!std::isfinite(cu) || !std::isfinite(cv)) return fail(GS_ERR_INVALID_ARG, "cube values must be finite");
    hipError_t e = gs::launch_init_box(s->p.storage, s->buf[s->parity][0], s->buf[s->parity][1], s->p.nx, s->p.ny,
                                       s->p.nz, x0, y0, z0, side, cu, cv, s->stream);
    return e == hipSuccess ? GS_OK : hip_fail(e, "fill kernel launch");
}

size_t gs_sqdiff_workspace_bytes(void) { return (size_t)gs::sqdiff_blocks() * sizeof(double); }

gs_status gs_sqdiff(const void *a, const void *b, size_t n, int32_t storage, void *workspace, void *hip_stream,
                    double *out)
{
    if (!a || !b || !workspace || !out) return fail(GS_ERR_INVALID_ARG, "NULL pointer");
    if (storage_bytes(storage) == 0) return fail(GS_ERR_INVALID_ARG, "unknown storage type %d", storage);
    if (!aligned(workspace, 8)) return fail(GS_ERR_INVALID_ARG, "workspace must be 8-byte aligned");
    hipStream_t st = (hipStream_t)hip_stream;
    std::vector<double> part(gs::sqdiff_blocks());
    hipError_t e = gs::launch_sqdiff(storage, a, b, n, (double *)workspace, st);
    if (e == hipSuccess) e = hipMemcpyAsync(part.data(), workspace, part.size() * 8, hipMemcpyDeviceToHost, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    if (e != hipSuccess) return hip_fail(e, "gs_sqdiff");
    double sum = 0.0;
    for (double x : part) sum += x;
    *out = sum;
    return GS_OK;
}

gs_status gs_laplacian7(const double *f, double *out, int32_t nx, int32_t ny, int32_t nz, void *hip_stream)
{
    if (!f || !out) return fail(GS_ERR_INVALID_ARG, "NULL pointer");
    if (!aligned(f, 256) || !aligned(out, 256)) return fail(GS_ERR_INVALID_ARG, "pointers must be 256-byte aligned");
    if (f == out) return fail(GS_ERR_INVALID_ARG, "in-place Laplacian is not supported");
    if (nx < 4 || ny < 4 || nz < 4 || nx % 8 != 0)
        return fail(GS_ERR_UNSUPPORTED, "grid %dx%dx%d unsupported (>= 4 each, nx %% 8 == 0)", nx, ny, nz);
    hipError_t e = gs::launch_laplacian7(f, out, nx, ny, nz, (hipStream_t)hip_stream);
    if (e != hipSuccess) return hip_fail(e, "laplacian launch");
    return GS_OK;
}

gs_status gs_copy(const void *src, void *dst, size_t bytes, void *hip_stream)
{
    if (!src || !dst) return fail(GS_ERR_INVALID_ARG, "NULL pointer");
    if (bytes % 16 != 0) return fail(GS_ERR_INVALID_ARG, "bytes must be a multiple of 16");
    if (!aligned(src, 16) || !aligned(dst, 16)) return fail(GS_ERR_INVALID_ARG, "pointers must be 16-byte aligned");
    if (bytes == 0) return GS_OK;
    hipError_t e = gs::launch_copy(src, dst, bytes, (hipStream_t)hip_stream);
    if (e != hipSuccess) return hip_fail(e, "copy launch");
    return GS_OK;
}

} // extern "C"
