// Device-side building blocks of the Gray-Scott kernels for gfx950:
// storage-type conversion, Philox4x32-10 noise, FP64 division by 6, and the
// Laplacians and the Euler step that all stencil kernels share.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace gs {

// ---------------------------------------------------------------- storage
struct bf16 {
    uint16_t bits;
};
typedef _Float16 f16;

__device__ __forceinline__ float to_f32(float x) { return x; }
__device__ __forceinline__ float to_f32(f16 x) { return (float)x; }
__device__ __forceinline__ float to_f32(bf16 x) { return __uint_as_float((uint32_t)x.bits << 16); }

// Round-to-nearest-even FP32 -> BF16 (NaN stays NaN): one gfx950
// conversion instruction.
__device__ __forceinline__ bf16 bf16_rne(float f)
{
    bf16 r;
    r.bits = __builtin_bit_cast(uint16_t, (__bf16)f);
    return r;
}

// Compute type C and conversions for each storage type S.
template <typename S> struct Traits;
template <> struct Traits<double> {
    typedef double C;
    static __device__ __forceinline__ double load(double s) { return s; }
    static __device__ __forceinline__ double store(double c) { return c; }
};
template <> struct Traits<float> {
    typedef float C;
    static __device__ __forceinline__ float load(float s) { return s; }
    static __device__ __forceinline__ float store(float c) { return c; }
};
template <> struct Traits<bf16> {
    typedef float C;
    static __device__ __forceinline__ float load(bf16 s) { return to_f32(s); }
    static __device__ __forceinline__ bf16 store(float c) { return bf16_rne(c); }
};
// BF16 storage with u kept as its complement 1 - u (v as it is). Most of a
// Gray-Scott state sits near u = 1, where BF16 steps are 2^-8 and the small
// updates of a step are rounded away; 1 - u is near 0 there and BF16 keeps
// eight significant bits of it. The same 2 bytes per value.
struct bf16c {
    uint16_t bits;
};
template <> struct Traits<bf16c> {
    typedef float C;
    static __device__ __forceinline__ float load(bf16c s) { return __uint_as_float((uint32_t)s.bits << 16); }
    static __device__ __forceinline__ bf16c store(float c)
    {
        bf16c r;
        r.bits = __builtin_bit_cast(uint16_t, (__bf16)c);
        return r;
    }
};
template <typename S> struct Complemented {
    static constexpr bool value = false;
};
template <> struct Complemented<bf16c> {
    static constexpr bool value = true;
};

template <> struct Traits<f16> {
    typedef float C;
    static __device__ __forceinline__ float load(f16 s) { return (float)s; }
    // The empty asm hides the FP32 value before the conversion (no
    // instruction): without it the compiler may fuse the conversion into the
    // fma that produced the value (an fma_mix with an FP16 result), which
    // rounds differently from the fma and then the conversion, and does so in
    // some kernels and not in others.
    static __device__ __forceinline__ f16 store(float c)
    {
        asm("" : "+v"(c));
        return (f16)c;
    }
};

// V consecutive storage elements moved as one aligned vector access.
template <typename S, int V> struct alignas(16) Vec {
    S e[V];
};

// ---------------------------------------------------------------- Philox
// Philox4x32-10 (Salmon et al., SC'11): 10 rounds; each multiplies counter
// words 0 and 2 by the round multipliers into 64-bit products and recombines
// (hi(M1 c2) ^ c1 ^ k0, lo(M1 c2), hi(M0 c0) ^ c3 ^ k1, lo(M0 c0)); the key is
// advanced by the two Weyl increments between rounds. The key and the step
// words are uniform across the launch.
struct Philox4 {
    uint32_t w[4];
};

// a ^ b ^ c in one instruction (gfx950 three-input bit operation; truth
// table 0x96 is the odd-parity function).
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c)
{
    return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}

__device__ __forceinline__ Philox4 philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                                 uint32_t k0, uint32_t k1)
{
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        // One 32x32 -> 64-bit multiply instruction per product (hi and lo together).
        const uint64_t pa = (uint64_t)0xD2511F53u * c0;
        const uint64_t pb = (uint64_t)0xCD9E8D57u * c2;
        c0 = xor3((uint32_t)(pb >> 32), c1, k0);
        c1 = (uint32_t)pb;
        c2 = xor3((uint32_t)(pa >> 32), c3, k1);
        c3 = (uint32_t)pa;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    Philox4 o;
    o.w[0] = c0; o.w[1] = c1; o.w[2] = c2; o.w[3] = c3;
    return o;
}

// r = (w + 1/2) 2^-31 for the signed word w: exact in FP64, in (-1, 1).
__device__ __forceinline__ double noise_word_f64(uint32_t w)
{
    return ((double)(int32_t)w + 0.5) * 0x1p-31;
}
// FP32 noise term n r = (n 2^-31) w + n 2^-32 for the signed word w, as one
// fma of the word converted to FP32 with the FP32 scales s = RN(n 2^-31),
// h = RN(n 2^-32) (the word keeps 24 significant bits, below what FP32
// storage resolves in the step).
__device__ __forceinline__ float noise_term_f32(uint32_t w, float s, float h)
{
    return __builtin_fmaf((float)(int32_t)w, s, h);
}

// The FP32 step's coefficients. Most kernels hold them in vector registers: on
// gfx950 an FP32 add, multiply or fma whose operands are vector registers or
// constants issues every 2.5 clocks per SIMD, and every 4.3 with a scalar register
// among them (measured, two or more waves per SIMD).
struct CoefF32 {
    float Du6, Dv6, F, FK, dt; // Du / 6, Dv / 6
    float ns, nh;              // noise 2^-31, noise 2^-32
};
__device__ __forceinline__ float in_vgpr(float x)
{
    asm volatile("" : "+v"(x)); // no instruction: the value is no longer known to be uniform
    return x;
}
// In scalar registers, for kernels that the number of their wavefronts or their
// spills bind more than the issue rate.
template <typename A> __device__ __forceinline__ CoefF32 coef_f32_scalar(const A &a)
{
    return CoefF32{a.Du6_f, a.Dv6_f, a.F_f, a.FK_f, a.dt_f, a.noise_s_f, a.noise_h_f};
}
template <typename A> __device__ __forceinline__ CoefF32 coef_f32(const A &a)
{
    return CoefF32{in_vgpr(a.Du6_f), in_vgpr(a.Dv6_f), in_vgpr(a.F_f),      in_vgpr(a.FK_f),
                   in_vgpr(a.dt_f),  in_vgpr(a.noise_s_f), in_vgpr(a.noise_h_f)};
}

// One Euler step of a cell in FP32 arithmetic (storage other than FP64):
// Eq. 1a/1b and 2a/2b with the products fused into the sums, so each field
// takes three operations after u v^2. lu6 and lv6 are six times the
// Laplacians, nr is the noise term n r (NOISE). Every FP32 kernel uses this
// one sequence, so results do not depend on the kernel, the tile or the fused
// depth.
template <bool NOISE>
__device__ __forceinline__ void euler_f32(const CoefF32 &k, float uc, float vc, float lu6, float lv6, float nr,
                                          float &uo, float &vo)
{
    const float uvv = uc * (vc * vc);
    float du = __builtin_fmaf(k.F, 1.0f - uc, __builtin_fmaf(k.Du6, lu6, -uvv));
    if constexpr (NOISE) du = du + nr;
    const float dv = __builtin_fmaf(-k.FK, vc, __builtin_fmaf(k.Dv6, lv6, uvv));
    uo = __builtin_fmaf(du, k.dt, uc);
    vo = __builtin_fmaf(dv, k.dt, vc);
}

// Noise of the 4 cells idx4 .. idx4+3 (idx4 a multiple of 4) at step t.
__device__ __forceinline__ Philox4 noise_block(uint64_t idx4, uint64_t t, uint64_t seed)
{
    const uint64_t q = idx4 >> 2;
    return philox4x32_10((uint32_t)q, (uint32_t)(q >> 32), (uint32_t)t, (uint32_t)(t >> 32),
                         (uint32_t)seed, (uint32_t)(seed >> 32));
}

// The same for block q < 2^32 (cells 4 q .. 4 q + 3 of a grid of less than 2^34
// cells): with the counter's second word 0 and the step words uniform, one of
// the two products is uniform in each of the first two rounds and runs on the
// scalar unit (36 instead of 40 vector instructions, and 32-bit indices).
__device__ __forceinline__ Philox4 noise_block32(uint32_t q, uint64_t t, uint64_t seed)
{
    return philox4x32_10(q, 0u, (uint32_t)t, (uint32_t)(t >> 32), (uint32_t)seed, (uint32_t)(seed >> 32));
}

// ---------------------------------------------------------------- arithmetic
// Correctly rounded x / 6 without the FP64 divide sequence: the IEEE
// quotient, bit for bit, for every finite x (a zero gives +0).
//
// With h = RN(1/6) and q0 = RN(x h), the residual r = x - 6 q0 is a small
// multiple of ulp(q0) (|r| <= 3 ulp(q0) and a little) and so exact in one
// fma, and x / 6 = q0 + r / 6. The quotient is RN(q0 + r c) for any c close
// enough to 1/6, except on an exact tie:
//  - Away from ties. x is an integer multiple of an ulp at least four times
//    the quotient's (x / 6 < x / 4), and of 2^-1074 where the quotient is
//    subnormal, so x / 6 sits at a multiple of 1/6 of the quotient's grid
//    step from a grid point and at least 1/6 of a step from every rounding
//    boundary. r (c - 1/6) moves it by at most 3 |c - 1/6| steps, far less
//    for |c - 1/6| <= 2^-23.
//  - Ties. Only a subnormal quotient can lie exactly half-way between two
//    grid points (x an odd multiple of 3 2^-1074); q0 is one of the two and
//    r = +-3 steps. RN(q0 + r c) is q0 for c below 1/6 and the other point
//    for c above it, while the rule wants the even one.
// So c is taken just below 1/6 when q0's last significand bit is 0 and just
// above it when that bit is 1: its high word is 0x3FC55555 and its low word
// the same constant with q0's last bit moved to bit 31 (0x3FC55555 or
// 0xBFC55555, both within 2^-24 of 1/6), one shift-or. The same constant in
// both words lets one register serve as the shift-or's operand and as the
// multiplier's high half. A tiny negative x gives RN(-0 + r c) = -0, as the
// division does.
// A numerator of +-Inf (an infinite input, or a neighbour sum beyond the
// largest double) gives NaN where the division gives +-Inf.
__host__ __device__ __forceinline__ double div6(double x)
{
    const double h = 0x1.5555555555555p-3; // RN(1/6), just below 1/6
    const double q0 = x * h;
    const double r = __builtin_fma(-q0, 6.0, x);
    const uint32_t k = 0x3FC55555u;
    const uint32_t lo = ((uint32_t)__builtin_bit_cast(uint64_t, q0) << 31) | k;
    const double c = __builtin_bit_cast(double, ((uint64_t)k << 32) | lo);
    return __builtin_fma(r, c, q0);
}

// Field-aware conversions between storage and compute values (field 0 is u,
// field 1 is v): the complemented storage type stores 1 - u. In FP32 1 - u is
// exact for u in [1/2, 2], and the stored complement of a u below 1/2 (at
// least 1/2) is rounded far more finely than by the storage.
template <typename S> __device__ __forceinline__ typename Traits<S>::C fload(int f, S s)
{
    const typename Traits<S>::C c = Traits<S>::load(s);
    if constexpr (Complemented<S>::value) return f == 0 ? 1.0f - c : c;
    else return c;
}
template <typename S> __device__ __forceinline__ S fstore(int f, typename Traits<S>::C c)
{
    if constexpr (Complemented<S>::value) return Traits<S>::store(f == 0 ? 1.0f - c : c);
    else return Traits<S>::store(c);
}

// Four values of field f to storage; BF16 converts them in pairs (one
// instruction each).
template <typename S> __device__ __forceinline__ Vec<S, 4> fstore4(int f, const typename Traits<S>::C (&c)[4])
{
    Vec<S, 4> r;
    if constexpr (sizeof(S) == 2 && !__is_same(S, f16)) {
        typedef float f2 __attribute__((ext_vector_type(2)));
        typedef __bf16 b2 __attribute__((ext_vector_type(2)));
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            f2 x = {c[2 * p], c[2 * p + 1]};
            if constexpr (Complemented<S>::value)
                if (f == 0) x = f2{1.0f - x[0], 1.0f - x[1]};
            const uint32_t w = __builtin_bit_cast(uint32_t, __builtin_convertvector(x, b2));
            r.e[2 * p].bits = (uint16_t)w;
            r.e[2 * p + 1].bits = (uint16_t)(w >> 16);
        }
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) r.e[e] = fstore<S>(f, c[e]);
    }
    return r;
}

// Six times the FP32-arithmetic Laplacian (the kernels' coefficients carry the
// 1/6). 2-byte storage: the neighbour sum less 6 c in FP32. Values of at most
// 11 significant bits whose exponents lie within 10 of each other (16 - 3 bits
// for BF16) add without any rounding, the fused 6 c included; beyond that each
// of the six roundings is within 2^-24 of the partial sum, while the state is
// rounded to 2^-9 (BF16) or 2^-12 (FP16) of itself after every step. Six
// operations against eleven for the sum of the differences n_i - c.
__device__ __forceinline__ float lap6_sum_f32(float c, float xm, float xp, float ym, float yp, float zm, float zp)
{
    return __builtin_fmaf(-6.0f, c, ((xm + xp) + (ym + yp)) + (zm + zp));
}
// Complemented BF16 storage: u = 1 - s carries the bits of a small s, which a
// sum near 6 would round away, so the differences n_i - c (of values near 1,
// exact) are summed.
__device__ __forceinline__ float lap6_diff_f32(float c, float xm, float xp, float ym, float yp, float zm, float zp)
{
    return ((xm - c) + (xp - c)) + ((ym - c) + (yp - c)) + ((zm - c) + (zp - c));
}
// FP32 storage: the sum less 6 c in FP64, which errs by at most 6 2^-53 of the
// summed magnitudes, rounded once to FP32. Converting each value (a row's cells
// serve as centre and as x-neighbours) takes 5.5 conversions and 6 operations
// per cell; converting the six differences took 6 and 11, and rounded each
// difference to FP32 first.
__device__ __forceinline__ float lap6_wide_f32(float c, float xm, float xp, float ym, float yp, float zm, float zp)
{
    const double s = (((double)xm + (double)xp) + ((double)ym + (double)yp)) + ((double)zm + (double)zp);
    return (float)__builtin_fma(-6.0, (double)c, s);
}
template <typename S>
__device__ __forceinline__ float lap6_f32(float c, float xm, float xp, float ym, float yp, float zm, float zp)
{
    if constexpr (Complemented<S>::value) return lap6_diff_f32(c, xm, xp, ym, yp, zm, zp);
    else if constexpr (sizeof(S) == 2) return lap6_sum_f32(c, xm, xp, ym, yp, zm, zp);
    else return lap6_wide_f32(c, xm, xp, ym, yp, zm, zp);
}

// FP64 Laplacian in the canonical order: ((x- + x+) + (y- + y+)) + (z- + z+),
// then (sum - 6 c) / 6.
__host__ __device__ __forceinline__ double lap_f64(double c, double xm, double xp, double ym, double yp,
                                                   double zm, double zp)
{
    const double s = ((xm + xp) + (ym + yp)) + (zm + zp);
    const double c6 = 6.0 * c;
    return div6(s - c6);
}

__device__ __forceinline__ int wrap(int i, int n) { return i < 0 ? i + n : (i >= n ? i - n : i); }

// Block index -> logical tile index such that the blocks the dispatcher
// sends to one XCD (hardware block ids congruent mod 8) get one contiguous
// range of logical tiles, so halos and z-chunk edges are shared in that
// XCD's L2.
__device__ __forceinline__ uint32_t xcd_logical_block(uint32_t b, uint32_t nb)
{
    const uint32_t per = nb >> 3;
    if (b >= (per << 3)) return b;
    return (b & 7u) * per + (b >> 3);
}

} // namespace gs
