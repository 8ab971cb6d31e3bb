// FP32 products on the FP16 matrix cores (gfx950).
//
// v_mfma_f32_16x16x4f32 does 1/16 of the products per cycle of
// v_mfma_f32_16x16x32_f16, so the wide FP32 sketches write both operands as sums of
// FP16 numbers and multiply those (every FP16 x FP16 product is exact, sums
// are FP32):
//   Omega: y = omega 2^13, b0 = fp16(y), b1 = fp16((y - b0) 2^11), b2 the rest of
//     (y - b0) 2^11: three terms hold the 24 significant bits exactly for |omega| >= 2^-25
//     and to within 2^-49 below;
//   A: x = a s with s a power of two, a0 = fp16(x), a1 = fp16(x - a0): 22 to 24
//     significant bits (|x - a0 - a1| <= 2^-23 |x|, at least 2^-25);
//   A Omega s 2^13 = sum a1 b0 + (a0 2^-11) b2 + (a0 2^-11) b1 + a0 b0, the
//     dropped a1 (b1 + b2) being at most 2^-22 of each product, of either sign.
// So a strip sum is within 2^-21 sum |a omega| + 2^-35 max|a| sum |omega| + 2^-49 sum |a| of
// the products' sum, besides the rounding of the additions.  The last two terms matter only
// where Omega brings out a row's small entries; a stored Omega that could is multiplied by
// the FP32 instruction instead (stored_columns), and so are strips narrower than a chunk.
// Relative Frobenius error against FP64 (N(0,1) A): 5.2e-7 to 5.4e-7 at 16384 to 32768
// columns, against 8.1e-7 of the FP32 instruction's chain of 512 additions per strip;
// 3.5e-7 against 5.7e-7 at 1024, equal at 16 to 31; 2.0e-7 against 1.2e-7 on rows with 2%
// of non-zeros.
// Time, k = 64 on 65536 x 16384: 854 us against 1219; k = 256 on 32768^2: 2.19 ms
// against 4.71; column-major k = 64 on 32768^2: 804 us against 1245.
// FP16 has 40 binades, so every row of A carries its own scale s: a strip's rows
// start from the largest |a| of their first non-zero chunk, put in [2^10, 2^11),
// and a row whose scaled entries pass 2^15 in a later chunk is scaled down again
// together with its sums (an exact power of two).  s depends on the row's
// entries and the chunk boundaries only, so a row's sums do not depend on m, the
// tile, the N-tile count or the storage order of A.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "sk_device.hpp"

#pragma clang fp contract(off)

namespace sk {

typedef _Float16 h2 __attribute__((ext_vector_type(2)));
typedef _Float16 h4 __attribute__((ext_vector_type(4)));
typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kSplitKC = 32;            // contraction columns per chunk = K of the MFMA
constexpr int kOmegaExp = 13;           // Omega's scale 2^13: |omega| <= 6 stays below FP16's 65504
constexpr int kLoExp = 11;              // b1, b2 are held 2^11 up, against a0 2^-11
constexpr int kRowExp = 10;             // largest scaled |a| of a row's first chunk: [2^10, 2^11)
constexpr float kRowLimit = 0x1p15f;    // scaled |a| past this rescales the row
constexpr float kRowStart = 0x1p127f;   // scale of a row that has been zero so far
// LDS row of one sketch column of a chunk: b0, b1, b2 of 32 contraction columns and 32
// bytes of padding (16-byte reads of 16 rows are free of bank conflicts at pitches of
// 2 mod 4 16-byte units, measured; at 13 units k = 256 on 32768^2 took 0.4% longer)
constexpr int kSplitRow = 3 * kSplitKC + 16;

// Omega value -> (b0, b1, b2); sc = 2^kOmegaExp.
__device__ __forceinline__ void split_omega(float z, float sc, _Float16& b0, _Float16& b1,
                                            _Float16& b2) {
    const float y = z * sc;
    b0 = (_Float16)y;
    const float r = (y - (float)b0) * 0x1p11f;
    b1 = (_Float16)r;
    b2 = (_Float16)(r - (float)b1);
}

// Four consecutive contraction columns kl .. kl + 3 (a multiple of 4) of a sketch
// column's LDS row.
__device__ __forceinline__ void split_store4(_Float16* row, int kl, const f32x4 z, float sc) {
    h4 b0, b1, b2;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        _Float16 x0, x1, x2;
        split_omega(z[u], sc, x0, x1, x2);
        b0[u] = x0;
        b1[u] = x1;
        b2[u] = x2;
    }
    *reinterpret_cast<h4*>(row + kl) = b0;
    *reinterpret_cast<h4*>(row + kSplitKC + kl) = b1;
    *reinterpret_cast<h4*>(row + 2 * kSplitKC + kl) = b2;
}

__device__ __forceinline__ void split_store1(_Float16* row, int kl, float z, float sc) {
    split_omega(z, sc, row[kl], row[kSplitKC + kl], row[2 * kSplitKC + kl]);
}

// max(m, largest |y| of 8 scaled values); NaN entries are passed over: their row's sums
// are NaN whatever the scale.
__device__ __forceinline__ float absmax8(const float (&y)[8], float m) {
#pragma unroll
    for (int e = 0; e < 8; e += 2)
        asm("v_max3_f32 %0, %0, |%1|, |%2|" : "+v"(m) : "v"(y[e]), "v"(y[e + 1]));
    return m;
}

// New scale of a row whose chunk holds the values x (8 per lane; the row's 32 in the
// lanes l, l ^ 16, l ^ 32, l ^ 48): s unchanged unless a scaled value passes the limit.
// Returns the factor 2^.. for the row's sums; an infinite entry sets `inf`.
__device__ __forceinline__ float rescale_row(const float (&x)[8], float& s, bool& inf) {
    uint32_t rm = 0;
#pragma unroll
    for (int e = 0; e < 8; ++e) rm = max(rm, __float_as_uint(x[e]) & 0x7FFFFFFFu);
    rm = max(rm, (uint32_t)__shfl_xor((int)rm, 16));
    rm = max(rm, (uint32_t)__shfl_xor((int)rm, 32));
    if (rm >= 0x7F800000u) {
        // infinity: the row is evaluated again at the end (a NaN's row is NaN anyway)
        inf = inf || rm == 0x7F800000u;
        if (s == kRowStart) s = 1.0f;
        return 1.0f;
    }
    if (!(__uint_as_float(rm) * s > kRowLimit)) return 1.0f;
    // exponent fields: 2^(kRowExp - E) for E the exponent of the largest entry (normal:
    // a subnormal never passes the limit)
    const int es = min(max(127 + kRowExp - ((int)(rm >> 23) - 127), 1), 254);
    const float f = __builtin_ldexpf(1.0f, es - (int)(__float_as_uint(s) >> 23));
    s = __uint_as_float((uint32_t)es << 23);
    return f;
}

// 8 scaled values -> the MFMA operands a0, a1 and a0 2^-11.
__device__ __forceinline__ void split_a(const float (&y)[8], h8& a0, h8& a1, h8& a0s) {
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        const f32x2 v = {y[2 * p], y[2 * p + 1]};
        const h2 h = __builtin_convertvector(v, h2);
        const f32x2 r = {v[0] - (float)h[0], v[1] - (float)h[1]};
        const h2 l = __builtin_convertvector(r, h2);
        a0[2 * p] = h[0];
        a0[2 * p + 1] = h[1];
        a1[2 * p] = l[0];
        a1[2 * p + 1] = l[1];
    }
    a0s = a0 * (_Float16)0x1p-11f;
}

// The four products of one chunk for one 16 x 16 tile of Y^T (Omega as the A operand,
// A as the B operand): small terms first.
__device__ __forceinline__ f32x4 split_mfma(const h8 b0, const h8 b1, const h8 b2, const h8 a0,
                                            const h8 a1, const h8 a0s, f32x4 acc) {
    acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(b0, a1, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(b2, a0s, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(b1, a0s, acc, 0, 0, 0);
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(b0, a0, acc, 0, 0, 0);
}

// Sum of a row with scale s -> its value.
__device__ __forceinline__ float unscale(float v, float s) {
    const int es = (int)(__float_as_uint(s) >> 23) - 127;
    return __builtin_ldexpf(v, -kOmegaExp - es);
}

}  // namespace sk
