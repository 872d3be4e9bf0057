// Internal interface of the surrogate network kernels (gs_surrogate.hip).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace gs {
namespace nn {

// Input normalisation of the (F, k) channels.
constexpr float F_CENTER = 0.035f, F_SCALE = 0.025f;
constexpr float K_CENTER = 0.055f, K_SCALE = 0.015f;

enum { MODE_HIDDEN = 0, MODE_OUT = 1, MODE_DGRAD = 2, MODE_ACT = 3 };

struct Geo {
    int nx, ny, nz;
    int ncell; // nx * ny * nz
};

struct ConvArgs {
    Geo geo;
    int nsamp;
    int zc;                 // planes per workgroup (set by the launcher)
    const uint16_t *in;     // channels-last BF16 input (CIN channels)
    const uint16_t *wpack;  // packed BF16 weights (B fragments)
    const float *bias;      // MODE_HIDDEN / MODE_ACT / MODE_OUT
    uint16_t *zout;         // MODE_HIDDEN: pre-activation (32 channels)
    uint16_t *aout;         // MODE_HIDDEN / MODE_ACT: activation; MODE_DGRAD: gradient (32 channels)
    const uint16_t *zprev;  // MODE_DGRAD: pre-activation of the layer below
    const void *res_u, *res_v; // MODE_OUT: residual input (planar, sample-major)
    void *out_u, *out_v;       // MODE_OUT: prediction (planar)
};

struct WgradArgs {
    Geo geo;
    int nsamp;
    const uint16_t *dz;  // output gradient, COUTS channels
    const uint16_t *act; // layer input, CIN channels
    int zc;              // first and last layers: planes per work item (set by the launcher)
    float *part;         // wgrad_blocks() x 27 x (16 MT) x (16 NT) partial sums (at least 1024 x 112 x 32 values)
    float *bpart;        // wgrad_blocks() x 32 partial sums of dz (bias gradient)
};

// (cus: compute units of the device)
hipError_t launch_conv(int cin, int mode, int io_f64, const ConvArgs &a, int cus, hipStream_t st);
int wgrad_blocks();
hipError_t launch_wgrad(const WgradArgs &a, hipStream_t st); // 32 -> 32 layers
// Weight and bias gradients of the first layer (8 stored input channels) or the
// last (8 stored output channels), from the tensors in `a`.
hipError_t launch_wgrad_edge(bool first, const WgradArgs &a, float *gW, float *gb, int cus, hipStream_t st);
hipError_t launch_wgrad_reduce(const float *part, float *gW, hipStream_t st);
hipError_t launch_bias_reduce(const float *bpart, float *gb, hipStream_t st); // 32 channels
// The samples' (F, k) go with the launch, up to FK_PER_LAUNCH samples at once:
// no device copy of them to wait for (a prediction at 128^3 lost 35 us to it).
constexpr int FK_PER_LAUNCH = 64;
struct FkArgs {
    float f[FK_PER_LAUNCH], k[FK_PER_LAUNCH];
};
hipError_t launch_pack_input(int io_f64, const void *u, const void *v, const FkArgs &fk, int nsamp, int ncell,
                             uint16_t *x, hipStream_t st);
int loss_blocks();
hipError_t launch_loss_grad(const float *pu, const float *pv, const float *tu, const float *tv, size_t rows,
                            float scale, uint16_t *dz4, double *part, hipStream_t st);
hipError_t launch_adam(float *p, const float *g, float *m, float *v, int n, float lr, float b1, float b2, float eps,
                       float c1, float c2, hipStream_t st);
// The output layer's forward weights (conv_out_kernel's order, 6 x 512 values).
hipError_t launch_repack_out(const float *W, uint16_t *out, hipStream_t st);
hipError_t launch_repack(const float *W, int cout, int cin, int cins, int nch, int dgrad, int lo_pairs, uint16_t *out,
                         hipStream_t st);

} // namespace nn
} // namespace gs
