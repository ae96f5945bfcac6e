// Exact sums of products modulo a prime below 2^50 in fp64, and the balanced form of their operands.
#pragma once
#include "ckks_internal.h"

namespace ckks {

// Sums of products in two doubles per output, without a reduction per product:
//   H' = fma(x, w, H)   with H held between 2^102 and 2^103, so that the product is rounded to a multiple of 2^50,
//   l  = fma(x, w, -(H' - H))   the rounded-off part, an exact integer, |l| <= 2^49,   L += l.
// 8 products of balanced operands (each at most 2^98 - 2^60), or 4 of a balanced and a canonical one (2^99 - 2^60), keep H
// in its binade from 1.5 * 2^102 and |L| below 2^52 + 2^51; fold() then
// moves H into L modulo q: with c = rint((H + L)/q), H - c q is an exact integer below 2^53, and the new |L| is below
// 1.1 q.  4 instructions per product and 6 per 8 products, against 7 and 3 with a quotient per product.
constexpr double MAC_H0 = 1.5 * 5070602400912917605986812821504.0;    // 1.5 * 2^102
struct MacSum {
    double h, l;
    __device__ __forceinline__ void mac(double x, double w) {
        const double n = fma(x, w, h);
        l += fma(x, w, h - n);
        h = n;
    }
    __device__ __forceinline__ void fold(double q, double u) {
        const double s = h - MAC_H0;
        const double c = rint(fma(s, u, l * u));
        l = fma(-c, q, s) + l;
        h = MAC_H0;
    }
    __device__ __forceinline__ u64 canonical(double q, double u) const {
        double v = fma(-rint(l * u), q, l);
        if (v < 0) v += q;
        return (u64)__double_as_longlong(v + 4503599627370496.0) & 0x000fffffffffffffull;
    }
};

// residue below 2^50 -> the balanced double of the same class
__device__ __forceinline__ u64 balanced_bits(u64 x, u64 q) {
    return (u64)__double_as_longlong((double)(int64_t)(x > q / 2 ? x - q : x));
}

// canonical residue below 2^52 -> the same integer as a double
__device__ __forceinline__ double canonical_double(u64 x) {
    return __longlong_as_double((long long)(x | 0x4330000000000000ull)) - 4503599627370496.0;
}

}  // namespace ckks
