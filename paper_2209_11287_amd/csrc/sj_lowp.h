// Rounding to the low-precision tiles' inputs and their proven band, shared by
// the block kernels (sj_lowp.hip, whose file comment has the derivation) and the
// hit-list count (sj_hits.hip).
#pragma once

#include <hip/hip_runtime.h>

namespace sj {

enum { PREC_F32 = 0, PREC_BF16 = 1, PREC_BF16X3 = 2, PREC_FP8 = 3 };

// FP32 -> BF16, round to nearest even (finite inputs).
__device__ __forceinline__ unsigned short f32_to_bf16(float f) {
    unsigned u = __float_as_uint(f);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (unsigned short)(u >> 16);
}
__device__ __forceinline__ float bf16_to_f32(unsigned short h) { return __uint_as_float(((unsigned)h) << 16); }

// FP64 -> FP8 E4M3 (the OCP "e4m3fn" form the gfx950 FP8 MFMA reads: bias
// 7, 3 mantissa bits, largest finite 448, subnormals down to 2^-9), rounded
// to nearest even in one step; |y| must be below 464 (the range guard keeps
// the scaled values far below). Returns the rounded value and its bits.
__device__ __forceinline__ double fp8_round(double y, unsigned &bits) {
    const double ay = fabs(y);
    const unsigned sign = y < 0.0 ? 0x80u : 0u;
    if (ay == 0.0) {
        bits = 0u;
        return 0.0;
    }
    const int e = ilogb(ay);
    const double spacing = e < -6 ? 0x1p-9 : ldexp(1.0, e - 3);
    const double q = rint(ay / spacing) * spacing;  // exact quotient (power of two), RNE
    unsigned code = 0u;
    if (q != 0.0) {
        const int eq = ilogb(q);
        if (eq < -6) code = (unsigned)(q * 0x1p9);  // subnormal: exponent field 0
        else code = ((unsigned)(eq + 7) << 3) | ((unsigned)(q * ldexp(1.0, 3 - eq)) - 8u);
    }
    bits = code ? (sign | code) : 0u;
    return sign ? -q : q;
}

// Rounds an FP64 value to the tile precision; returns the rounded value as
// a double (exact) and its storage bits (split BF16: hi in the low half, lo
// in the high half; the value is hi + lo).
template <int PREC>
__device__ __forceinline__ double round_in(double y, unsigned &bits) {
    if constexpr (PREC == PREC_FP8) return fp8_round(y, bits);
    const float f = (float)y;  // RNE
    if (PREC == PREC_F32) {
        bits = __float_as_uint(f);
        return (double)f;
    }
    const unsigned short h = f32_to_bf16(f);
    const float fh = bf16_to_f32(h);
    if (PREC == PREC_BF16) {
        bits = h;
        return (double)fh;
    }
    const unsigned short l = f32_to_bf16(f - fh);  // f - fh exact
    bits = (unsigned)h | ((unsigned)l << 16);
    return (double)fh + (double)bf16_to_f32(l);
}

__device__ __forceinline__ double gam(double m, double u) { return m * u / (1.0 - m * u); }

// Band half-width of one query row (see the file comment), in the scaled
// units of the tiles (eps in [1, 2)): a2 = |q'|^2. Besides the relative
// terms, FP32 / BF16 values below the normal range (2^-126) may be flushed:
// at most 2^-126 per coordinate (2^-123 per vector of d <= 64) on the inputs
// and 2^-126 per product or partial sum, norm and threshold conversion.
template <int PREC>
__device__ __forceinline__ double lp_delta(double a2, double eps, double eps2, int d, int K) {
    const double u64 = 0x1p-53, u32 = 0x1p-24;
    // input rounding unit: FP32; BF16 via FP32 (two roundings); split BF16:
    // |fl32(y) - hi| <= 2^-8 |fl32(y)| and lo rounds that to 2^-8 of itself
    // (FP8: relative 2^-4 for normal values, from FP64 in one rounding)
    const double uin = PREC == PREC_F32    ? 0x1p-24
                       : PREC == PREC_BF16 ? (0x1p-8 + 0x1p-24)
                       : PREC == PREC_FP8  ? 0x1p-4
                                           : (0x1p-16 + 0x1p-24 + 0x1p-39);
    const double eta = uin + u64 + uin * u64;
    const double ua = 2.0 * 0x1p-24;
    const double a = sqrt(a2 * (1.0 + 1e-12));
    const double epsp = eps * (1.0 + (d + 4) * u64);
    // FP8 subnormals: at most 2^-10 per coordinate, 2^-7 per vector of d <= 64, for q' and c'
    const double e = eta * (2.0 * a + epsp) / (1.0 - 2.0 * eta) + 0x1p-122 +
                     (PREC == PREC_FP8 ? 0x1p-6 : 0.0);  // conversion error at |c'| = a + tau
    const double tau = epsp + e;
    const double b = a + tau;  // candidates beyond cannot be near the threshold
    const double A2 = a * a, B2 = b * b;
    // split BF16: 3d non-zero products per tile (the zero padding adds
    // exactly); sum_k (|hi|+|lo|)(|hi|+|lo|) over both rows is at most
    // (1 + 2^-6)^2 |q'||c'|, and the dropped 2 sum_k lo_q lo_c at most
    // 2 (2^-8 (1 + 2^-6))^2 |q'||c'| <= 2^-14 a b
    const int nt = PREC == PREC_BF16X3 ? 3 * d : K;
    const double gk = gam(nt + 1, ua);
    const double sp = PREC == PREC_BF16X3 ? (1.0 + 0x1p-6) * (1.0 + 0x1p-6) : 1.0;
    const double drop = PREC == PREC_BF16X3 ? 0x1p-14 : 0.0;
    const double F = (u32 + gam(d, u64) + gk) * B2 + (2.0 * gk * sp + drop) * a * b  // accumulation
                     + gam(d, u64) * A2 + u32 * (eps2 + A2)                        // threshold
                     + (2.0 * nt + 16.0) * 0x1p-126;                               // flushed tiny values
    return 2.0 * (F + 2.0 * tau * e + e * e + gam(d + 2, u64) * tau * tau) + (d + 2) * 0x1p-1021;
}

}  // namespace sj
