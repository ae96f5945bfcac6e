// Hybrid key switching for rot / conj (Table 1) with the input-side work hoisted.
//
// The paper treats rot and conj as primitives and says nothing about how they
// are evaluated; this is the standard RNS hybrid method with dnum digits:
//   decompose:  INTT(c1) -> per digit D_j approximate base conversion of
//               [c1]_{Q_Dj} to every other active limb and to the special
//               primes (ModUp) -> NTT.  Done ONCE per ciphertext.
//   switch:     per Galois element g: u = sum_j sigma_g(d_j) (.) key_j over the
//               level+K limbs (the automorphism is an index gather in the NTT
//               domain, fused into the loads) -> INTT of the K special limbs ->
//               base conversion P -> Q, subtract, times P^-1 (ModDown) ->
//               + sigma_g(c0).
// Base conversions use no floating-point correction term.  Sums of products modulo primes below 2^50 are kept in two
// doubles and folded every few products (mac_device.h), modulo larger primes in 128 bits; either is reduced once.
#include <algorithm>

#include "ckks_internal.h"
#include "common_kernels.h"
#include "mac_device.h"
#include "ntt_device.h"

namespace ckks {

constexpr u32 KS_THREADS = EW_THREADS;
constexpr u32 DN_CHUNK = 24;   // target limbs per workgroup in ModDown (2, 3, 4, 6, 12, 24 measured: fewer, larger groups are faster)

__device__ __forceinline__ u32 galois_index(u32 k, u32 g, u32 logN) {
    // entry k holds the value at psi^(2*bitrev(k)+1); sigma_g reads the value at that exponent times g
    u32 e = 2u * (__brev(k) >> (32 - logN)) + 1u;
    u32 e2 = (e * g) & ((2u << logN) - 1u);
    return __brev((e2 - 1u) >> 1) >> (32 - logN);
}

// Entries k, k + 1 (k even) of sigma_g of a row: their exponents differ by N, and g is odd, so their sources do too: they are
// entries kp and kp ^ 1, kp = galois_index(k).  PAIR: one 16-byte load gives them in memory order, turned() puts them in the
// order asked for; the kernels turn a pair where they use it (turned as it is loaded, every load is waited for on its own:
// passb_final_kernel 602 us per 24 switches against 525 turned where used and 537 with two 8-byte loads).  Otherwise: two
// 8-byte loads in the order asked for, which a launch of few workgroups, bound by the latency of one of them, has sooner.
typedef u64 pair_t __attribute__((ext_vector_type(2)));
template <bool PAIR>
__device__ __forceinline__ pair_t load_two(const u64 *__restrict__ row, u32 kp) {
    return PAIR ? *reinterpret_cast<const pair_t *>(row + (kp & ~1u)) : pair_t{row[kp], row[kp ^ 1u]};
}
template <bool PAIR>
__device__ __forceinline__ pair_t turned(pair_t v, u32 kp) { return PAIR && (kp & 1) ? pair_t{v[1], v[0]} : v; }

// Evaluation keys as the library holds them: rows of ciphertext limbs carry the factor P^-1 of ModDown (the base
// conversion P -> q_i carries it too, so that no kernel after the key product multiplies by it), on primes below 2^50 as
// balanced doubles, on others in Montgomery form; rows of special limbs are in Montgomery form.  In place if in == out.
// rows [rows][N], row r modulo limb r % W; four residues per thread (one per thread leaves too few bytes in flight: a
// 25 MB key took 34 us longer).  grid: x = 1024 residues (N >= 1024), y = row
__global__ __launch_bounds__(EW_THREADS) void key_form_kernel(const u64 *in, u64 *out,
                                                              const ModConst *__restrict__ mods,
                                                              const u64 *__restrict__ pinv, u32 L, u32 W, u32 N) {
    const u32 limb = blockIdx.y - uniform_div(blockIdx.y, W) * W;
    const ModConst m = mods[limb];
    const u64 f = limb < L ? pinv[limb] : 0;
    const size_t idx = (size_t)blockIdx.y * N + (blockIdx.x * EW_THREADS + threadIdx.x) * 2;
    pair_t v[2];
#pragma unroll
    for (u32 h = 0; h < 2; ++h) v[h] = *reinterpret_cast<const pair_t *>(in + idx + h * (N / 2));
#pragma unroll
    for (u32 h = 0; h < 2; ++h) {
#pragma unroll
        for (u32 e = 0; e < 2; ++e) {
            const u64 x = limb < L ? mont_mul(v[h][e], f, m) : v[h][e];
            v[h][e] = limb < L && (m.q >> 50) == 0 ? balanced_bits(x, m.q) : mont_mul(x, m.r2, m);
        }
        *reinterpret_cast<pair_t *>(out + idx + h * (N / 2)) = v[h];
    }
}

struct PtrPack {
    const u64 *p[ROT_BATCH];
};

// tmp[r][i][n] = src_r[i][n]: collects the c1 halves of up to ROT_BATCH ciphertexts
__global__ __launch_bounds__(KS_THREADS) void gather_c1_kernel(PtrPack src, u64 *__restrict__ tmp, u32 level, u32 N) {
    const u32 n = blockIdx.x * KS_THREADS + threadIdx.x;
    const u32 i = blockIdx.y, r = blockIdx.z;
    tmp[((size_t)r * level + i) * N + n] = src.p[r][(size_t)i * N + n];
}

// The same collection fused with the first pass of the inverse transform (rings with the two-pass kernels):
// reads the c1 halves where they are, writes tmp[r][i] half transformed.  grid: x = 4096-residue tiles,
// y = r * level + i.
template <u32 RL>
__global__ __launch_bounds__(Tile<RL>::THREADS) void gather_intt_kernel(PtrPack src, u64 *__restrict__ tmp,
                                                                  const ModConst *__restrict__ mods,
                                                                  const ModFp *__restrict__ modf,
                                                                  const u64 *__restrict__ tw,
                                                                  const double *__restrict__ twf,
                                                                  const u64 *__restrict__ ninv, u32 level, u32 logN) {
    __shared__ u64 lds[Tile<RL>::WORDS];
    const u32 r = uniform_div(blockIdx.y, level), i = blockIdx.y - r * level;
    const u64 *in = src.p[r] + ((size_t)i << logN);
    u64 *out = tmp + ((size_t)blockIdx.y << logN);
    auto load = [&](u32 idx) { return in[idx]; };
    auto store = [&](u32 idx, u64 v) { out[idx] = v; };
    with_field(modf[i], mods, tw, twf, ninv, i, logN, [&](const auto &f) { pass_b_body<true, RL>(f, logN, lds, load, store); });
}

// (out0, out1, t2) = (a0 b0, a0 b1 + a1 b0, a1 b1), pointwise, and the inverse tile pass of t2, which the relinearisation
// decomposes: t2 as it is and, half transformed, tmp.  As two kernels a product and rescale at 2^15 (12 + 4 primes) took 4.5 us
// longer: a launch, and 64-bit Montgomery products where primes below 2^50 have cheaper ones.  Where they have not, a workgroup is a
// chain of those products and of the butterflies, and below 2^15 the launch costs less than that: a product on primes of 61 bits, one
// kernel / two, 2^12, 2 limbs 50.5 / 49.7, 6 59.4 / 58.4, 2^13, 12 100.4 / 98.5, 2^14, 12 123.2 / 121.5 us, of 52 bits 47.5 / 46.9, 56.9 /
// 55.8, 93.7 / 92.5, 117.5 / 116.6, of 58 as those; 2^15, 12 limbs of 61 / 58 / 52 bits 114.3 / 110.5 / 107.9 and 115.2 / 112.1 / 109.0,
// 2^16, 24 of 52 234 and 237.  Of 50 bits: 2^12, 6 33.6 and 34.1, 2^14, 12 93.7 and 94.8, 2^15, 12 61.5 and 64.8.
// grid: x = 4096-residue tiles, y = limb
template <u32 RL>
__global__ __launch_bounds__(Tile<RL>::THREADS) void tensor_intt_kernel(const u64 *__restrict__ a, const u64 *__restrict__ b,
                                                                  u64 *__restrict__ out, u64 *__restrict__ t2,
                                                                  u64 *__restrict__ tmp, const ModConst *__restrict__ mods,
                                                                  const ModFp *__restrict__ modf,
                                                                  const u64 *__restrict__ tw,
                                                                  const double *__restrict__ twf,
                                                                  const u64 *__restrict__ ninv, u32 level, u32 logN) {
    typedef Tile<RL> TL;
    __shared__ u64 lds[TL::WORDS];
    const u32 i = blockIdx.y, tid = threadIdx.x;
    const size_t row = ((size_t)i << logN) + (blockIdx.x << 12), half = (size_t)level << logN;
    u64 *dst = tmp + ((size_t)i << logN);
    auto store = [&](u32 idx, u64 v) { dst[idx] = v; };
    const ModFp mf = modf[i];
    auto pointwise = [&](auto products) {
#pragma unroll
        for (u32 e0 = 0; e0 < TL::R; e0 += 4) {                     // four residues' operands on their way together
            u64 x[4][4];
#pragma unroll
            for (u32 e = 0; e < 4; ++e) {
                const size_t k = row + TL::one(tid, e0 + e);
                x[e][0] = a[k];
                x[e][1] = a[half + k];
                x[e][2] = b[k];
                x[e][3] = b[half + k];
            }
#pragma unroll
            for (u32 e = 0; e < 4; ++e) {
                const u32 loc = TL::one(tid, e0 + e);
                u64 r0, r1, r2;
                products(x[e][0], x[e][1], x[e][2], x[e][3], r0, r1, r2);
                out[row + loc] = r0;
                out[half + row + loc] = r1;
                t2[row + loc] = r2;
                lds[TL::slot(loc)] = r2;
            }
        }
    };
    if (mf.ok) {
        const FieldFp f = make_field_fp(mf, twf, i, logN);
        pointwise([&](u64 a0, u64 a1, u64 b0, u64 b1, u64 &r0, u64 &r1, u64 &r2) {
            const double x0 = f.in(a0), x1 = f.in(a1), y0 = f.in(b0), y1 = f.in(b1);
            r0 = f.out(f.mul(x0, y0));
            r1 = f.out(f.mul(x0, y1) + f.mul(x1, y0));
            r2 = f.out(f.mul(x1, y1));
        });
        pass_b_inv_from_lds<RL>(f, logN, lds, store);
    } else {
        const ModConst m = mods[i];
        pointwise([&](u64 a0, u64 a1, u64 b0, u64 b1, u64 &r0, u64 &r1, u64 &r2) {
            b0 = mont_mul(b0, m.r2, m);
            b1 = mont_mul(b1, m.r2, m);
            r0 = mont_mul(a0, b0, m);
            r1 = add_mod(mont_mul(a0, b1, m), mont_mul(a1, b0, m), m.q);
            r2 = mont_mul(a1, b1, m);
        });
        with_int_field(mf, mods, tw, ninv, i, logN, [&](const auto &f) { pass_b_inv_from_lds<RL>(f, logN, lds, store); });
    }
}

// Per ciphertext r and digit j: y_i = c_i * (Q_D/q_i)^-1 mod q_i for the limbs of the digit, then for
// every target t outside the digit out_t = sum_i y_i * (Q_D/q_i mod t) mod t (coefficient domain).
// Targets inside the digit are left out: in the NTT domain they are the input's own rows, which the consumers
// read in place (no copy, no transform).
// grid: x = pairs of coefficients, y = digit, z = ciphertext; targets t0 .. t1-1.  A thread owns two
// adjacent coefficients (16-byte accesses) so that every conversion factor, which is workgroup-uniform and
// arrives through the scalar cache, serves two multiply-accumulates; AMAX bounds the digit size.
template <u32 AMAX, u32 VEC, bool FP>
__global__ __launch_bounds__(KS_THREADS) void modup_kernel(const u64 *__restrict__ c1_coeff,
                                                           u64 *__restrict__ digits,
                                                           const ModConst *__restrict__ mods,
                                                           const ModFp *__restrict__ modf,
                                                           const u64 *__restrict__ up_inv,
                                                           const u64 *__restrict__ up_mat,
                                                           const u64 *__restrict__ up_matf, u32 level, u32 K, u32 L,
                                                           u32 alpha, u32 N, u32 beta, u32 t0, u32 t1) {
    typedef u64 vec_t __attribute__((ext_vector_type(2)));
    const u32 n = (blockIdx.x * KS_THREADS + threadIdx.x) * VEC;
    const u32 j = blockIdx.y;
    const u32 r = blockIdx.z;
    const u32 Wl = level + K;
    const u32 lo = j * alpha, hi = min(lo + alpha, level);
    const u64 *coef = c1_coeff + (size_t)r * level * N;
    u64 *dig = digits + (size_t)r * beta * Wl * N;
    u64 y[AMAX][VEC];
#pragma unroll
    for (u32 a = 0; a < AMAX; ++a) {
#pragma unroll
        for (u32 e = 0; e < VEC; ++e) y[a][e] = 0;
        if (lo + a < hi) {
            const u64 inv = up_inv[lo + a];
            const ModConst m = mods[lo + a];
#pragma unroll
            for (u32 e = 0; e < VEC; e += 2) {
                const vec_t c = *reinterpret_cast<const vec_t *>(coef + (size_t)(lo + a) * N + n + e);
                y[a][e] = mont_mul(c[0], inv, m);
                y[a][e + 1] = mont_mul(c[1], inv, m);
            }
        }
    }
    if (FP) {
        // Every prime involved is below 2^50 (the launcher checks): y is exact in a double, every product is
        // split exactly into h + l and brought below 0.9 q before it is added, and the partial sum is reduced
        // every four terms (below 2^53).  Twice the multiply rate of the 32-bit integer pipeline.
        double yd[AMAX][VEC];
#pragma unroll
        for (u32 a = 0; a < AMAX; ++a)
#pragma unroll
            for (u32 e = 0; e < VEC; ++e) yd[a][e] = (double)y[a][e];
        for (u32 t = t0; t < t1; ++t) {
            if (t >= lo && t < hi) continue;      // the digit's own limbs: consumers read them from the source
            u64 *dst = dig + ((size_t)j * Wl + t) * N + n;
            const double q = modf[t].q, u = modf[t].u;
            double fd[AMAX], acc[VEC];
#pragma unroll
            for (u32 a = 0; a < AMAX; ++a)
                fd[a] = lo + a < hi ? __longlong_as_double((long long)up_matf[(size_t)(lo + a) * Wl + t]) : 0.0;
#pragma unroll
            for (u32 e = 0; e < VEC; ++e) acc[e] = 0.0;
#pragma unroll
            for (u32 a = 0; a < AMAX; ++a) {
#pragma unroll
                for (u32 e = 0; e < VEC; ++e) {
                    const double h = yd[a][e] * fd[a], l = fma(yd[a][e], fd[a], -h);
                    acc[e] += fma(-rint(h * u), q, h) + l;
                    if ((a & 3) == 3) acc[e] = fma(-rint(acc[e] * u), q, acc[e]);
                }
            }
#pragma unroll
            for (u32 e = 0; e < VEC; e += 2) {
                vec_t o;
#pragma unroll
                for (u32 z = 0; z < 2; ++z) {
                    double v = fma(-rint(acc[e + z] * u), q, acc[e + z]);
                    if (v < 0) v += q;
                    o[z] = (u64)v;
                }
                *reinterpret_cast<vec_t *>(dst + e) = o;
            }
        }
    } else {
        for (u32 t = t0; t < t1; ++t) {
            if (t >= lo && t < hi) continue;
            u64 *dst = dig + ((size_t)j * Wl + t) * N + n;
            const u32 gl = t < level ? t : L + (t - level);
            u64 f[AMAX];
#pragma unroll
            for (u32 a = 0; a < AMAX; ++a) f[a] = lo + a < hi ? up_mat[(size_t)(lo + a) * Wl + t] : 0;
            u128 acc[VEC];
#pragma unroll
            for (u32 e = 0; e < VEC; ++e) acc[e] = {0, 0};
#pragma unroll
            for (u32 a = 0; a < AMAX; ++a)        // a factor of 0 pads digits shorter than AMAX
#pragma unroll
                for (u32 e = 0; e < VEC; ++e) mac(acc[e], y[a][e], f[a]);
            const ModConst mt = mods[gl];
#pragma unroll
            for (u32 e = 0; e < VEC; e += 2) {
                vec_t o;
                o[0] = redc_wide(acc[e], mt);     // up to AMAX products below 2^62 * q each
                o[1] = redc_wide(acc[e + 1], mt);
                *reinterpret_cast<vec_t *>(dst + e) = o;
            }
        }
    }
}

// The base conversions of the two fused kernels below sum products of 32 x 32-bit multiply-adds, which run at the rate of fp64
// ones here (31e12 per second, both) and are exact in 64 bits instead of 53: a source limb costs a target 4 of them, where exact
// sums in doubles take 6 (60-bit sources, or targets of 60 bits; two-double sums 4), three times the factor bytes and twice
// the registers, so that a thread's two coefficients now share each factor.  us before and after: moddown_mid_kernel of a bank
// of 27 switches at 2^16 406 and 350, with the rescale (9 blocks) 150 and 118, one switch 25.2 and 21.3; modup_mid_kernel of 32
// ciphertexts of 24 limbs 467 and 421, one of 17 37.8 and 30.1, three of 2^15 (11 limbs) 57.7 and 50.1.
//
// The two BITS-bit pieces of the source limbs' values of a coefficient:
template <u32 KM, u32 BITS>
__device__ __forceinline__ void mid_pieces(const u64 (&yraw)[KM], u32 (&yp)[KM][2]) {
#pragma unroll
    for (u32 k = 0; k < KM; ++k) {
        yp[k][0] = (u32)yraw[k] & ((1u << BITS) - 1);
        yp[k][1] = (u32)(yraw[k] >> BITS);
    }
}

// hi 2^25 + lo mod q (below 2^50) as a double, at most q + 2^32; hi and lo below 2^60
__device__ __forceinline__ double mid_reduce(u64 lo, u64 hi, double q, double u) {
    const double t1 = fma((double)(u32)(hi >> 32), 33554432.0, (double)(u32)(lo >> 32)) * 4294967296.0;
    const double t2 = (double)(u32)hi * 33554432.0;
    return (fma(-rint(t1 * u), q, t1) + fma(-rint(t2 * u), q, t2)) + (double)(u32)lo;
}

// sum_k y_k F_k mod q (below 2^50) as a double, at most q + 2^32: the pieces (at most 30 bits) times the factors F_k 2^(BITS a)
// mod q in 25-bit halves, 16 products of 55 bits.  The sums' words then become doubles: hi 2^25 + lo = (hh 2^25 + lh) 2^32 +
// hl 2^25 + ll, the first two terms exact (52 and 32 significant bits) and reduced one by one.
template <u32 KM>
__device__ __forceinline__ double mid_convert(const u32 (&yp)[KM][2], const u32 *__restrict__ f, double q, double u) {
    u64 lo = 0, hi = 0;
#pragma unroll
    for (u32 k = 0; k < KM; ++k) {
#pragma unroll
        for (u32 a = 0; a < 2; ++a) {
            lo += (u64)yp[k][a] * f[(k * 2 + a) * 2 + 0];
            hi += (u64)yp[k][a] * f[(k * 2 + a) * 2 + 1];
        }
    }
    return mid_reduce(lo, hi, q, u);
}

// The same sums at N = 2^12, where a tile pass is a whole transform and a base conversion needs no columns: the workgroup that
// transforms a target row forms it, residue by residue of its first round, from the n rows of canonical y behind one another at
// `rows` (four residues of four rows on their way together).  done(j, s0, s1): the two sums of the j-th residue, of BITS-bit
// pieces; f: the target's factors, 4 words a source row.  Conversions as launches of their own took 3 to 4 us each, three in a
// switch and rescale, and their rows a write and a read: the toy projection (2^12, two batches of switches) 110.5 -> 95.7 us.
template <u32 RL, u32 BITS, class Done>
__device__ __forceinline__ void tile_convert(const u64 *__restrict__ rows, u32 n, const u32 *__restrict__ f, Done done) {
    constexpr u32 R = 1u << RL, G = 4;
#pragma unroll
    for (u32 j0 = 0; j0 < R; j0 += G) {
        u64 s0[G], s1[G];
#pragma unroll
        for (u32 j = 0; j < G; ++j) s0[j] = s1[j] = 0;
        for (u32 k0 = 0; k0 < n; k0 += 4) {
            u64 y[4][G];
#pragma unroll
            for (u32 k = 0; k < 4; ++k)
#pragma unroll
                for (u32 j = 0; j < G; ++j) y[k][j] = k0 + k < n ? rows[(size_t)(k0 + k) * 4096 + Round<RL, 0>::elem(j0 + j)] : 0;
#pragma unroll
            for (u32 k = 0; k < 4; ++k) {
                if (k0 + k >= n) break;
                const u32 *fk = f + (k0 + k) * 4;
#pragma unroll
                for (u32 j = 0; j < G; ++j) {
                    const u32 lo = (u32)y[k][j] & ((1u << BITS) - 1), hi = (u32)(y[k][j] >> BITS);
                    s0[j] += (u64)lo * fk[0];
                    s1[j] += (u64)lo * fk[1];
                    s0[j] += (u64)hi * fk[2];
                    s1[j] += (u64)hi * fk[3];
                }
            }
        }
#pragma unroll
        for (u32 j = 0; j < G; ++j) done(j0 + j, s0[j], s1[j]);
    }
}

// ModUp at N = 2^12: conversion and transform of a target row in one workgroup.  y [n][level][N]: canonical c1 (Q_D/q_i)^-1 in
// the coefficient domain; digits as modup_mid_kernel's, transformed.  Needs what that kernel needs.
// grid: x = row of the extended basis, y = digit, z = ciphertext
template <u32 RL>
__global__ __launch_bounds__(Tile<RL>::THREADS) void modup_tile_kernel(const u64 *__restrict__ y, u64 *__restrict__ digits,
                                                                 const ModConst *__restrict__ mods,
                                                                 const ModFp *__restrict__ modf,
                                                                 const double *__restrict__ twf_fwd,
                                                                 const u64 *__restrict__ tws_fwd,
                                                                 const u64 *__restrict__ ninvs,
                                                                 const u32 *__restrict__ up_ft,
                                                                 const u32 *__restrict__ up_mats, u32 level, u32 K, u32 L,
                                                                 u32 alpha, u32 am, u32 beta) {
    typedef Tile<RL> TL;
    __shared__ u64 lds[TL::WORDS];
    const u32 t = blockIdx.x, j = blockIdx.y, r = blockIdx.z, Wl = level + K;
    const u32 lo = j * alpha, nd = min(alpha, level - lo);
    if (t >= lo && t < lo + nd) return;                              // the digit's own limbs
    const u32 gl = t < level ? t : L + (t - level);
    const u64 *src = y + ((size_t)r * level + lo) * 4096;
    u64 *dst = digits + (((size_t)r * beta + j) * Wl + t) * 4096;
    const ModFp mf = modf[gl];
    u64 raw[TL::R];
    auto go = [&](const auto &f) {
        pass_b_fwd_from_regs<false, RL, true>(f, 12, lds, raw, 0);
#pragma unroll
        for (u32 i = 0; i < TL::R; ++i) dst[TL::one(threadIdx.x, i)] = lds[TL::slot(TL::one(threadIdx.x, i))];
    };
    if (t < level) {
        tile_convert<RL, 25>(src, nd, up_ft + ((size_t)j * Wl + t) * (am * 4), [&](u32 i, u64 s0, u64 s1) {
            raw[i] = (u64)__double_as_longlong(mid_reduce(s0, s1, mf.q, mf.u));
        });
        go(make_field_fp(mf, twf_fwd, gl, 12));
        return;
    }
    const u32 *f = up_mats + ((size_t)j * K + (t - level)) * (am * 4);
    if (mf.pm) {
        const FieldPm fp = make_field_pm(mods, tws_fwd, ninvs, gl, 12);
        tile_convert<RL, 25>(src, nd, f, [&](u32 i, u64 s0, u64 s1) { raw[i] = fp.fold30(s0, s1, false); });
        go(fp);
        return;
    }
    const ModConst m = mods[gl];
    tile_convert<RL, 25>(src, nd, f, [&](u32 i, u64 s0, u64 s1) {
        u128 acc{s0, 0};                                             // s0 + s1 2^30 < 2^90
        acc_add(acc, u128{s1 << 30, s1 >> 34});
        raw[i] = redc(acc, m);
        if (mf.ok) raw[i] = (u64)__double_as_longlong(canonical_double(raw[i]));
    });
    with_field(mf, mods, tws_fwd, twf_fwd, ninvs, gl, 12, go);
}

// Decomposition between the two tile passes at N = 2^(12+LOGR), one kernel instead of four.  The last LOGR stages of the
// inverse transform of c1, the base conversion of every digit (ModUp) and the first LOGR stages of the forward transform
// of the extended rows all work on columns (residues 4096 apart); a workgroup owns a tile of 1024 coefficients, 1024 >> LOGR
// columns of 2^LOGR rows, of one digit of one ciphertext:
//   1. wavefront a: the columns of limb lo + a of the digit in registers, last inverse round with
//      N^-1 (Q_D/q_i)^-1 folded in -> y_a in LDS;
//   2. every thread takes two coefficients of the tile, both at once for each target of a group of UP_TG (a target's factors
//      arrive once for both): exact sums of 25-bit pieces of y, onto the ciphertext primes by mid_convert, onto the special
//      primes with factors in 30-bit parts and one Montgomery reduction of the recombined 90-bit sum -> LDS;
//   3. wavefront t: the columns of target t from LDS, first forward round (fp64 or integer butterflies), out.
// A wavefront per row has the row's twiddles, modulus and addresses in scalar registers: 114 vector registers for digits of
// eight limbs, which two such workgroups per CU leave.  With 32 threads per row (tiles of 512 coefficients, 256 threads) it is
// 148 and 186 registers with the quotient and the folding butterflies, two or three wavefronts per SIMD for four.  32
// ciphertexts of 24 limbs, in a projection's giant step, 514 us so with quotients, 420 now; one of 17 limbs 28.2 and 24.9.
// At N = 2^12 (LOGR = 0; for consumers that transform the digits themselves) the tile passes are whole transforms, the inverse
// one carries the scaling, and a thread converts and stores its own coefficients, without LDS.
// c1_half [n][level][N]: c1 after the inverse tile pass; digits [n][beta][level+K][N]: rows of targets outside the
// digit, ready for the forward tile pass.  AM: the digit size alpha rounded up to a power of two; the factor tables are
// padded with zeros to it.  Needs alpha, K <= 8, every active ciphertext prime below 2^50 and every special prime below
// 2^60 (the launcher checks).  grid: x = column tile, y = digit, z = ciphertext.
// With its counterpart moddown_mid_kernel, against separate column passes and conversions: a ciphertext product and rescale
// at 2^15 (12 + 4 primes) 186 -> 159 us, a bank of 24 switches at 2^14 (level 5 of 6, 2 special primes) 257 -> 232 us.
// MidTile: the workgroup and tile of these kernels (2^12: no tile in LDS, small workgroups).
template <u32 LOGR>
struct MidTile {
    static constexpr u32 THREADS = LOGR ? 512 : 256, SIZE = 2 * THREADS, COLS = SIZE >> LOGR, PER = LOGR ? COLS / 64 : 0;
};
inline u32 mid_tile(const ckks_params *p) { return p->logN == 12 ? MidTile<0>::SIZE : MidTile<1>::SIZE; }
constexpr u32 UP_TG = 8;
template <u32 LOGR, u32 AM>
__global__ __launch_bounds__(MidTile<LOGR>::THREADS, 4) void modup_mid_kernel(const u64 *__restrict__ c1_half, u64 *__restrict__ digits,
                                                        const ModConst *__restrict__ mods,
                                                        const ModFp *__restrict__ modf,
                                                        const ModFp *__restrict__ modf_up,
                                                        const double *__restrict__ twf_inv,
                                                        const double *__restrict__ twf_fwd,
                                                        const u64 *__restrict__ tws_fwd,
                                                        const u64 *__restrict__ ninvs,
                                                        const u32 *__restrict__ up_ft,
                                                        const u32 *__restrict__ up_mats, u32 level, u32 K, u32 L,
                                                        u32 alpha, u32 beta, u32 tsplit, u32 tg) {
    typedef MidTile<LOGR> MT;
    constexpr u32 logN = 12 + LOGR, N = 1u << logN, R = 1u << LOGR, MID_TILE = MT::SIZE, COLS = MT::COLS, PER = MT::PER;
    static_assert(UP_TG == 8 && AM <= 8, "the target tiles reuse the 8 rows of source tiles");
    __shared__ u64 ylds[LOGR ? 8 * MID_TILE : 1];
    u64 *wlds = ylds;               // the sources live in registers once step 2 has read them: the same 64 KiB
    const u32 tid = threadIdx.x, lane = tid & 63, grp = __builtin_amdgcn_readfirstlane(tid / 64);   // grp < 8
    // tsplit > 1 (few ciphertexts): the groups of targets of a tile go to tsplit workgroups, each of which redoes
    // step 1, so that a lone decomposition still fills the chip
    const u32 tile = blockIdx.x % (N / MID_TILE), tpart = blockIdx.x / (N / MID_TILE);
    const u32 c0 = tile * COLS;
    const u32 j = blockIdx.y, r = blockIdx.z;
    const u32 Wl = level + K;
    const u32 lo = j * alpha, hi = min(lo + alpha, level), nd = hi - lo;
    u64 yraw[2][AM];
    if constexpr (LOGR == 0) {
#pragma unroll
        for (u32 a = 0; a < AM; ++a) {
            yraw[0][a] = yraw[1][a] = 0;
            if (a < nd) {
                const u64 *src = c1_half + ((size_t)r * level + lo + a) * N + c0 + tid;
#pragma unroll
                for (u32 e = 0; e < 2; ++e) yraw[e][a] = src[e * MT::THREADS];
            }
        }
    } else if (grp < nd) {
        const u32 i = lo + grp;
        const RowBuf src(c1_half + ((size_t)r * level + i) * N, N);
        const FieldFp f = make_field_fp(modf_up[i], twf_inv, i, logN);
#pragma unroll
        for (u32 c = 0; c < PER; ++c) {
            const u32 col = lane + 64 * c;
            auto load = [&](u32 at, u32) { return src.load(at + c0, col); };
            auto store = [&](u32 at, u32, u64 v) { ylds[grp * MID_TILE + (at >> 12) * COLS + col] = v; };
            pass_a_body<true, LOGR>(f, c0 + col, load, store);
        }
    }
    if constexpr (LOGR != 0) {
        __syncthreads();
#pragma unroll
        for (u32 e = 0; e < 2; ++e)
#pragma unroll
            for (u32 a = 0; a < AM; ++a) yraw[e][a] = a < nd ? ylds[a * MID_TILE + e * MT::THREADS + tid] : 0;
        __syncthreads();            // every thread has its y: the tile may be overwritten
    }
    u32 yp[2][AM][2];
#pragma unroll
    for (u32 e = 0; e < 2; ++e) mid_pieces<AM, 25>(yraw[e], yp[e]);
    u64 *dig = digits + ((size_t)r * beta + j) * Wl * N;
    const u32 nt = Wl - nd;                                          // targets: all rows outside the digit
    for (u32 u0 = tpart * tg; u0 < nt; u0 += tsplit * tg) {
        const u32 here = min(tg, nt - u0);
        for (u32 tt = 0; tt < UP_TG && tt < here; ++tt) {
            const u32 uu = u0 + tt, t = uu < lo ? uu : uu + nd;      // row of the extended basis
            u64 res[2];
            if (t < level) {
                // target among the ciphertext primes
                const double q = modf[t].q, u = modf[t].u;
                const u32 *f = up_ft + ((size_t)j * Wl + t) * (AM * 4);   // zero beyond the digit's limbs, as y is
#pragma unroll
                for (u32 e = 0; e < 2; ++e) {
                    const double v = mid_convert<AM>(yp[e], f, q, u);    // the forward round normalises it
                    if constexpr (LOGR == 0)
                        res[e] = make_field_fp(modf[t], twf_fwd, t, logN).out(v);
                    else
                        res[e] = (u64)__double_as_longlong(v);
                }
            } else {
                // target among the special primes: sum_a sum_b y_ab F_ab, F_ab = F_a 2^64 2^(25b) mod p in two 30-bit parts
                // (without the 2^64 on primes that fold, where the sum folds like a product does)
                const u32 k = t - level;
                const u32 *f = up_mats + ((size_t)j * K + k) * (AM * 4);
                const bool pm = modf[L + k].pm;
#pragma unroll
                for (u32 e = 0; e < 2; ++e) {
                    u64 s0 = 0, s1 = 0;                              // 16 products of 55 bits each
#pragma unroll
                    for (u32 a = 0; a < AM; ++a)
#pragma unroll
                        for (u32 b = 0; b < 2; ++b) {
                            s0 += (u64)yp[e][a][b] * f[(a * 2 + b) * 2 + 0];
                            s1 += (u64)yp[e][a][b] * f[(a * 2 + b) * 2 + 1];
                        }
                    if (pm) {
                        res[e] = make_field_pm(mods, tws_fwd, ninvs, L + k, logN).fold30(s0, s1, LOGR == 0);
                        continue;
                    }
                    u128 acc{s0, 0};                                 // s0 + s1 2^30 < 2^90
                    acc_add(acc, u128{s1 << 30, s1 >> 34});
                    res[e] = redc(acc, mods[L + k]);                 // canonical: the factors carry 2^64
                    if (LOGR != 0 && modf[L + k].ok) res[e] = (u64)__double_as_longlong(canonical_double(res[e]));
                }
            }
#pragma unroll
            for (u32 e = 0; e < 2; ++e) {
                if constexpr (LOGR == 0)
                    dig[(size_t)t * N + c0 + e * MT::THREADS + tid] = res[e];
                else
                    wlds[tt * MID_TILE + e * MT::THREADS + tid] = res[e];
            }
        }
        if constexpr (LOGR != 0) {
            __syncthreads();
            if (grp < here) {
                const u32 uu = u0 + grp, t = uu < lo ? uu : uu + nd;
                const u32 gl = t < level ? t : L + (t - level);
                const RowBuf dst(dig + (size_t)t * N, N);
                const ModFp mf = modf[gl];
#pragma unroll
                for (u32 c = 0; c < PER; ++c) {
                    const u32 col = lane + 64 * c;
                    if (mf.ok) {
                        const FieldFp ff = make_field_fp(mf, twf_fwd, gl, logN);
                        double v[R];
#pragma unroll
                        for (u32 jj = 0; jj < R; ++jj)
                            v[jj] = __longlong_as_double((long long)wlds[grp * MID_TILE + jj * COLS + col]);
                        radix_fwd<LOGR>(ff, v, 0, 0);
#pragma unroll
                        for (u32 jj = 0; jj < R; ++jj) dst.store(jj * 4096 + c0, col, ff.half(v[jj]));
                    } else {
                        auto load = [&](u32 at, u32) { return wlds[grp * MID_TILE + (at >> 12) * COLS + col]; };
                        auto store = [&](u32 at, u32, u64 v) { dst.store(at + c0, col, v); };
                        with_int_field(mf, mods, tws_fwd, ninvs, gl, logN,
                                       [&](const auto &f) { pass_a_body<false, LOGR>(f, c0 + col, load, store); });
                    }
                }
            }
            __syncthreads();
        }
    }
}

// the instance for a ring (N = 2^12 .. 2^16) and a digit size
typedef decltype(&modup_mid_kernel<4, 8>) modup_mid_t;
template <u32 LOGR>
static modup_mid_t modup_mid_for(u32 am) {
    return am == 1 ? modup_mid_kernel<LOGR, 1> : am == 2 ? modup_mid_kernel<LOGR, 2>
         : am == 4 ? modup_mid_kernel<LOGR, 4> : modup_mid_kernel<LOGR, 8>;
}
static modup_mid_t modup_mid_for(const ckks_params *p) {
    const u32 am = pad_pow2(p->alpha);
    switch (p->logN) {
        case 12: return modup_mid_for<0>(am);
        case 13: return modup_mid_for<1>(am);
        case 14: return modup_mid_for<2>(am);
        case 15: return modup_mid_for<3>(am);
        default: return modup_mid_for<4>(am);
    }
}

constexpr u32 MAX_BETA = 4;    // digits the fused kernels unroll (larger dnum uses the plain kernels)
constexpr u32 EPI = 4;         // residues whose loads are issued together in the fused kernels
constexpr u32 KEY_GROUP = 4;   // key switches that share one key are served by one thread

struct ItemPack {
    SwitchItem it[ROT_BATCH];
    uint8_t grp_first[ROT_BATCH], grp_count[ROT_BATCH];   // runs of items with the same key
};

// u[r][comp][t][k] = sum_j digits_r[j][t][sigma_g(k)] * key[j][comp][limb(t)][k] for the items r of one
// group (same key, same Galois element): each key residue is loaded once and used for all of them.
// grid: x = coefficients, y = limb t, z = group.
__global__ __launch_bounds__(KS_THREADS) void inner_product_kernel(ItemPack pack, u64 *__restrict__ u,
                                                                   const ModConst *__restrict__ mods, u32 level,
                                                                   u32 K, u32 L, u32 beta, u32 alpha, u32 logN) {
    const u32 N = 1u << logN;
    const u32 k = blockIdx.x * KS_THREADS + threadIdx.x;
    const u32 t = blockIdx.y;
    const u32 first = pack.grp_first[blockIdx.z], cnt = pack.grp_count[blockIdx.z];
    const u32 Wl = level + K, Wt = L + K;
    const u32 gl = t < level ? t : L + (t - level);
    const u64 *key = pack.it[first].key;
    const u32 kp = galois_index(k, (u32)pack.it[first].galois_elt, logN);
    const ModConst m = mods[gl];
    const bool fp = t < level && (m.q >> 50) == 0;               // keys of these rows are balanced doubles
    const double q = (double)m.q, uq = 1.0 / q;
    u128 a0[KEY_GROUP], a1[KEY_GROUP];
    MacSum f0[KEY_GROUP], f1[KEY_GROUP];
#pragma unroll
    for (u32 r = 0; r < KEY_GROUP; ++r) {
        a0[r] = a1[r] = {0, 0};
        f0[r] = f1[r] = MacSum{MAC_H0, 0.0};
    }
    for (u32 j = 0; j < beta; ++j) {
        const u64 k0 = key[(((size_t)j * 2 + 0) * Wt + gl) * N + k];
        const u64 k1 = key[(((size_t)j * 2 + 1) * Wt + gl) * N + k];
#pragma unroll
        for (u32 r = 0; r < KEY_GROUP; ++r) {
            if (r < cnt) {
                const SwitchItem &it = pack.it[first + r];
                const u64 d = (t < level && t / alpha == j) ? it.c1[(size_t)t * N + kp]
                                                            : it.digits[((size_t)j * Wl + t) * N + kp];
                if (fp) {
                    const double x = canonical_double(d);
                    f0[r].mac(x, __longlong_as_double((long long)k0));
                    f1[r].mac(x, __longlong_as_double((long long)k1));
                    if ((j & 3) == 3) {
                        f0[r].fold(q, uq);
                        f1[r].fold(q, uq);
                    }
                } else {
                    mac(a0[r], d, k0);
                    mac(a1[r], d, k1);
                }
            }
        }
    }
#pragma unroll
    for (u32 r = 0; r < KEY_GROUP; ++r) {
        if (r < cnt) {
            u64 *u0 = u + (((size_t)(first + r) * 2 + 0) * Wl + t) * N + k;
            u64 *u1 = u + (((size_t)(first + r) * 2 + 1) * Wl + t) * N + k;
            if (fp) {
                f0[r].fold(q, uq);
                f1[r].fold(q, uq);
                *u0 = f0[r].canonical(q, uq);
                *u1 = f1[r].canonical(q, uq);
            } else {
                *u0 = redc_wide(a0[r], m);
                *u1 = redc_wide(a1[r], m);
            }
        }
    }
}

// Inner products of several rotations summed in the extended basis (the merged giant step): a thread owns one
// coefficient of one limb for MR ciphertexts, so that a key residue, read once, serves MR multiply-accumulates.
// Rows of ciphertext primes below 2^50 (FP) sum in doubles, folded after each rotation's products; the others keep 128-bit
// sums, folded before more than 16 products (each below 2^124) have been added.  grid.y indexes `rows`, the rows of the
// extended basis this launch covers.
constexpr u32 MR = 3;
template <bool FP>
__global__ __launch_bounds__(KS_THREADS) void merged_ip_kernel(MergedRot rots, const u64 *__restrict__ digits,
                                                               size_t dig_w, const u64 *__restrict__ c0_base,
                                                               size_t c0_stride_r, u64 *__restrict__ dst_base,
                                                               size_t dst_stride, u64 *__restrict__ u,
                                                               const ModConst *__restrict__ mods, u32 n, u32 level,
                                                               u32 K, u32 L, u32 beta, u32 alpha, u32 logN,
                                                               u32 accumulate, u32 groups, LimbIds rows) {
    const u32 N = 1u << logN;
    // grid x = ((chunk of 8 coefficient runs) * groups + group of MR ciphertexts) * 8 + run within the chunk: the
    // groups of ciphertexts, which read the same key rows, follow each other at a distance of 8 workgroups, i.e. on
    // the same XCD at about the same time, so one of them fetches a key line and the others find it in that L2
    const u32 chunk = N / KS_THREADS < 8 ? N / KS_THREADS : 8;   // a power of two
    const u32 xg = uniform_div(blockIdx.x, chunk);
    const u32 xd = uniform_div(xg, groups);
    const u32 k = (xd * chunk + (blockIdx.x & (chunk - 1))) * KS_THREADS + threadIdx.x;
    const u32 t = rows.id[blockIdx.y];
    const u32 r0 = (xg - xd * groups) * MR;
    const u32 Wl = level + K, Wt = L + K;
    const u32 gl = t < level ? t : L + (t - level);
    const u32 own = t < level ? uniform_div(t, alpha) : ~0u;                 // the digit whose own limb t is: read from c1
    const ModConst m = mods[gl];
    const double q = (double)m.q, uq = 1.0 / q;
    u128 a0[MR], a1[MR];
    MacSum f0[MR], f1[MR];
    double csf[MR];
    u64 s0[MR], s1[MR], cs[MR];
#pragma unroll
    for (u32 r = 0; r < MR; ++r) {
        a0[r] = a1[r] = {0, 0};
        f0[r] = f1[r] = MacSum{MAC_H0, 0.0};
        s0[r] = s1[r] = cs[r] = 0;
        csf[r] = 0.0;
    }
    u32 terms = 0;
    for (u32 i = 0; i < rots.n_rot; ++i) {
        const u32 kp = galois_index(k, (u32)rots.galois_elt[i], logN);
        const u64 *key = rots.key[i];
        // the loads of up to MAX_BETA digits are issued before their products
        for (u32 j0 = 0; j0 < beta; j0 += MAX_BETA) {
            u64 k0[MAX_BETA], k1[MAX_BETA], d[MAX_BETA][MR];
#pragma unroll
            for (u32 jj = 0; jj < MAX_BETA; ++jj) {
                const u32 j = j0 + jj;
                if (j < beta) {
                    k0[jj] = key[(((size_t)j * 2 + 0) * Wt + gl) * N + k];
                    k1[jj] = key[(((size_t)j * 2 + 1) * Wt + gl) * N + k];
#pragma unroll
                    for (u32 r = 0; r < MR; ++r)
                        if (r0 + r < n)
                            d[jj][r] = own == j
                                           ? c0_base[(size_t)(r0 + r) * c0_stride_r + rots.c0_off[i] +
                                                     ((size_t)level + t) * N + kp]
                                           : digits[((size_t)i * n + r0 + r) * dig_w + ((size_t)j * Wl + t) * N + kp];
                }
            }
#pragma unroll
            for (u32 jj = 0; jj < MAX_BETA; ++jj)
                if (j0 + jj < beta) {
#pragma unroll
                    for (u32 r = 0; r < MR; ++r)
                        if (r0 + r < n) {
                            if (FP) {
                                const double x = canonical_double(d[jj][r]);
                                f0[r].mac(x, __longlong_as_double((long long)k0[jj]));
                                f1[r].mac(x, __longlong_as_double((long long)k1[jj]));
                            } else {
                                mac(a0[r], d[jj][r], k0[jj]);
                                mac(a1[r], d[jj][r], k1[jj]);
                            }
                        }
                }
            if (FP) {                                            // at most MAX_BETA = 4 products since the last fold
#pragma unroll
                for (u32 r = 0; r < MR; ++r) {
                    f0[r].fold(q, uq);
                    f1[r].fold(q, uq);
                }
            }
        }
        if (t < level) {
#pragma unroll
            for (u32 r = 0; r < MR; ++r)
                if (r0 + r < n) {
                    const u64 c = c0_base[(size_t)(r0 + r) * c0_stride_r + rots.c0_off[i] + (size_t)t * N + kp];
                    if (FP)
                        csf[r] += canonical_double(c);           // up to MERGE_GROUP = 8 residues: below 2^53
                    else
                        cs[r] = add_mod(cs[r], c, m.q);
                }
        }
        if (!FP) {
            terms += beta;
            if (terms + beta > 16 || i + 1 == rots.n_rot) {
#pragma unroll
                for (u32 r = 0; r < MR; ++r) {
                    s0[r] = add_mod(s0[r], redc_wide(a0[r], m), m.q);
                    s1[r] = add_mod(s1[r], redc_wide(a1[r], m), m.q);
                    a0[r] = a1[r] = {0, 0};
                }
                terms = 0;
            }
        }
    }
#pragma unroll
    for (u32 r = 0; r < MR; ++r) {
        if (r0 + r < n) {
            u64 *u0 = u + (((size_t)(r0 + r) * 2 + 0) * Wl + t) * N + k;
            u64 *u1 = u + (((size_t)(r0 + r) * 2 + 1) * Wl + t) * N + k;
            u64 v0 = s0[r], v1 = s1[r], c = cs[r];
            if (FP) {
                v0 = f0[r].canonical(q, uq);
                v1 = f1[r].canonical(q, uq);
                c = MacSum{0.0, csf[r]}.canonical(q, uq);
            }
            if (accumulate) {
                v0 = add_mod(v0, *u0, m.q);
                v1 = add_mod(v1, *u1, m.q);
            }
            *u0 = v0;
            *u1 = v1;
            if (t < level) {
                u64 *d = dst_base + (size_t)(r0 + r) * dst_stride + (size_t)t * N + k;
                *d = add_mod(*d, c, m.q);
            }
        }
    }
}

// The same sum straight from digits that still lack their forward tile pass (decompose with `half`): sigma_g moves whole
// tiles (the top bits of an index fix its exponent modulo 2N / 4096), so a workgroup that owns output tile T of row t of one
// ciphertext transforms, rotation by rotation and digit by digit, the one tile that sigma_g brings to T, in LDS, and takes
// its products from there: the transformed digits, each used once, never reach memory.
// Bound by the chain of a workgroup's loads, transform and gather (two workgroups of 512 threads per CU hide each other's)
// and by the integer butterflies of the special limbs.  RL = 3: eight residues a thread, whose sums, keys and transform fit
// the 128 registers that two workgroups leave (RL = 4 takes 200 and more; any spilling costs more than the fusion gives: 2.98
// ms where this took 1.81).  A digit's key loads are issued before the barrier in front of its products; the next digit
// loaded there as well spills or gains nothing.  QKV projection, 63 rotations of 24 + 8 limbs: 1.43 ms of tile passes and
// 1.04 of merged_ip_kernel before, 1.81 in one (the call 17.05 -> 16.38 ms), 1.58 with the folding butterflies.
template <u32 RL>
__global__ __launch_bounds__(Tile<RL>::THREADS, 4) void merged_tile_kernel(MergedRot rots, const u64 *__restrict__ digits,
                                                                        size_t dig_w, const u64 *__restrict__ c0_base,
                                                                        size_t c0_stride_r, u64 *__restrict__ dst_base,
                                                                        size_t dst_stride, u64 *__restrict__ u,
                                                                        const ModConst *__restrict__ mods,
                                                                        const ModFp *__restrict__ modf,
                                                                        const u64 *__restrict__ tw_fwd,
                                                                        const double *__restrict__ twf_fwd,
                                                                        const u64 *__restrict__ ninv, u32 n, u32 level,
                                                                        u32 K, u32 L, u32 beta, u32 alpha, u32 logN,
                                                                        u32 accumulate, LimbIds rows) {
    typedef Tile<RL> TL;
    constexpr u32 PP = TL::R / 2;
    __shared__ u64 lds[TL::WORDS];
    const u32 N = 1u << logN, Wl = level + K, Wt = L + K, tid = threadIdx.x;
    // units (row, tile) in chunks of eight, the ciphertexts of a unit eight workgroups apart: on one XCD at about the same
    // time, where one of them fetches the key lines for all.  Special limbs, the longest rows, first.
    const u32 tiles = N >> 12, xg = blockIdx.x >> 3, xn = uniform_div(xg, n), unit = xn * 8 + (blockIdx.x & 7), r = xg - xn * n;
    if (unit >= tiles * Wl) return;
    const u32 t = rows.id[unit >> (logN - 12)], tile = unit & (tiles - 1), base = tile << 12;
    const u32 gl = t < level ? t : L + (t - level);
    const u32 own = t < level ? uniform_div(t, alpha) : ~0u;                 // the digit whose own limb t is: read from c1
    const ModConst m = mods[gl];
    const ModFp mf = modf[gl];
    u64 *u0 = u + (((size_t)r * 2) * Wl + t) * N + base, *u1 = u0 + (size_t)Wl * N;
    auto tile_of = [&](u32 i) { return galois_index(base, (u32)rots.galois_elt[i], logN) >> 12; };
    auto go = [&](const auto &f, auto zero, auto mac, auto in, auto norm, auto out) {
        decltype(zero) a0[TL::R], a1[TL::R];
#pragma unroll
        for (u32 e = 0; e < TL::R; ++e) a0[e] = a1[e] = zero;
        u64 raw[TL::R];                                          // the next digit to transform, on its way
        auto fetch = [&](u32 i, u32 j) {
            const u64 *row = digits + ((size_t)i * n + r) * dig_w + ((size_t)j * Wl + t) * N + ((size_t)tile_of(i) << 12);
#pragma unroll
            for (u32 e = 0; e < TL::R; ++e) raw[e] = __builtin_nontemporal_load(row + Round<RL, 0>::elem(e));
        };
        for (u32 i = 0; i < rots.n_rot; ++i) {
            for (u32 j = 0; j < beta; ++j) {
                // opaque: twiddles and gather addresses kept over the digits would take the registers of another workgroup
                u32 g = (u32)rots.galois_elt[i], src_tile = tile_of(i);
                asm volatile("" : "+s"(src_tile), "+s"(g));
                const u64 *key = rots.key[i] + ((size_t)j * 2 * Wt + gl) * N + base;
                auto products = [&](u32 e, auto x0, auto x1, pair_t k0, pair_t k1) {
                    a0[2 * e] = mac(a0[2 * e], x0, k0[0]);
                    a1[2 * e] = mac(a1[2 * e], x0, k1[0]);
                    a0[2 * e + 1] = mac(a0[2 * e + 1], x1, k0[1]);
                    a1[2 * e + 1] = mac(a1[2 * e + 1], x1, k1[1]);
                };
                auto load0 = [&](u32 e) { return *reinterpret_cast<const pair_t *>(key + TL::pair(tid, e)); };
                auto load1 = [&](u32 e) { return *reinterpret_cast<const pair_t *>(key + (size_t)Wt * N + TL::pair(tid, e)); };
                if (j != own) {
                    fetch(i, j);
                    pass_b_fwd_from_regs<true, RL>(f, logN, lds, raw, src_tile);
                    pair_t k0[PP], k1[PP];
#pragma unroll
                    for (u32 e = 0; e < PP; ++e) {
                        k0[e] = load0(e);
                        k1[e] = load1(e);
                    }
                    __syncthreads();
#pragma unroll
                    for (u32 e = 0; e < PP; ++e) {
                        const u32 l = galois_index(base + TL::pair(tid, e), g, logN) & 4095;
                        products(e, f.from_bits(lds[TL::slot(l)]), f.from_bits(lds[TL::slot(l ^ 1)]), k0[e], k1[e]);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    __syncthreads();
                } else {
                    // the digit's own limb, transformed as it is; two pairs at a time, for the registers
                    const u64 *row = c0_base + (size_t)r * c0_stride_r + rots.c0_off[i] + ((size_t)level + t) * N;
#pragma unroll
                    for (u32 e0 = 0; e0 < PP; e0 += 2) {
                        pair_t k0[2], k1[2], d[2];
                        u32 kp[2];
#pragma unroll
                        for (u32 e = 0; e < 2; ++e) {
                            kp[e] = galois_index(base + TL::pair(tid, e0 + e), g, logN);
                            d[e] = load_two<true>(row, kp[e]);
                            k0[e] = load0(e0 + e);
                            k1[e] = load1(e0 + e);
                        }
#pragma unroll
                        for (u32 e = 0; e < 2; ++e) {
                            const pair_t v = turned<true>(d[e], kp[e]);
                            products(e0 + e, in(v[0]), in(v[1]), k0[e], k1[e]);
                        }
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
                if ((j & 3) == 3 || j + 1 == beta) {                // fp64: q/2 and four products below 0.9 q, under 2^53
#pragma unroll
                    for (u32 e = 0; e < TL::R; ++e) {
                        norm(a0[e]);
                        norm(a1[e]);
                    }
                }
            }
        }
#pragma unroll
        for (u32 e = 0; e < PP; ++e) {
            pair_t v0{out(a0[2 * e]), out(a0[2 * e + 1])}, v1{out(a1[2 * e]), out(a1[2 * e + 1])};
            pair_t *p0 = reinterpret_cast<pair_t *>(u0 + TL::pair(tid, e)), *p1 = reinterpret_cast<pair_t *>(u1 + TL::pair(tid, e));
            if (accumulate) {
                const pair_t o0 = *p0, o1 = *p1;
#pragma unroll
                for (u32 z = 0; z < 2; ++z) {
                    v0[z] = add_mod(v0[z], o0[z], m.q);
                    v1[z] = add_mod(v1[z], o1[z], m.q);
                }
            }
            *p0 = v0;
            *p1 = v1;
        }
    };
    if (mf.ok && t < level) {
        const FieldFp f = make_field_fp(mf, twf_fwd, gl, logN);
        go(f, 0.0, [&](double a, double x, u64 k) { return a + f.mul(x, __longlong_as_double((long long)k)); },
           [&](u64 x) { return canonical_double(x); }, [&](double &a) { f.norm(a); }, [&](double a) { return f.out(a); });
    } else if (mf.ok) {                                          // a special prime below 2^50
        const FieldFp f = make_field_fp(mf, twf_fwd, gl, logN);
        go(f, (u64)0, [&](u64 a, double x, u64 k) { return add_mod(a, mont_mul(f.out(x), k, m), m.q); },
           [&](u64 x) { return canonical_double(x); }, [&](u64 &) {}, [&](u64 a) { return a; });
    } else if (mf.pm) {
        const FieldPm f = make_field_pm(mods, tw_fwd, ninv, gl, logN);
        // x normalised, so x + q in (0, 2q)
        go(f, (u64)0, [&](u64 a, int64_t x, u64 k) { return add_mod(a, mont_mul((u64)x + m.q, k, m), m.q); },
           [&](u64 x) { return (int64_t)x; }, [&](u64 &) {}, [&](u64 a) { return a; });
    } else {
        const FieldInt f = make_field_int(mods, tw_fwd, ninv, gl, logN);
        // x as the butterflies leave it, below 4q <= 2^64: a product below q 2^64
        go(f, (u64)0, [&](u64 a, u64 x, u64 k) { return add_mod(a, mont_mul(x, k, m), m.q); }, [&](u64 x) { return x; },
           [&](u64 &) {}, [&](u64 a) { return a; });
    }
    if (t < level) {
        u64 cs[TL::R];
#pragma unroll
        for (u32 e = 0; e < TL::R; ++e) cs[e] = 0;
        for (u32 i = 0; i < rots.n_rot; ++i) {
            const u64 *row = c0_base + (size_t)r * c0_stride_r + rots.c0_off[i] + (size_t)t * N;
            pair_t d[PP];
            u32 kp[PP];
#pragma unroll
            for (u32 e = 0; e < PP; ++e) {
                kp[e] = galois_index(base + TL::pair(tid, e), (u32)rots.galois_elt[i], logN);
                d[e] = load_two<true>(row, kp[e]);
            }
#pragma unroll
            for (u32 e = 0; e < PP; ++e) {
                const pair_t v = turned<true>(d[e], kp[e]);
#pragma unroll
                for (u32 z = 0; z < 2; ++z) cs[2 * e + z] = add_mod(cs[2 * e + z], v[z], m.q);
            }
        }
        u64 *dst = dst_base + (size_t)r * dst_stride + (size_t)t * N + base;
#pragma unroll
        for (u32 e = 0; e < PP; ++e) {
            pair_t *p = reinterpret_cast<pair_t *>(dst + TL::pair(tid, e));
            const pair_t o = *p;
            *p = pair_t{add_mod(o[0], cs[2 * e], m.q), add_mod(o[1], cs[2 * e + 1], m.q)};
        }
    }
}

// y holds, per (item, component), the K special-limb rows y_k = INTT(u_{p_k}) * (P/p_k)^-1 in the coefficient
// domain (the scaling comes out of the inverse transform); row (pc, k) starts at y + (pc*ystride + yoff + k)*N.
// w_i = sum_k y_k * (P/p_k mod q_i) mod q_i for a chunk of target limbs i.
template <u32 KMAX, bool FP>
__global__ __launch_bounds__(KS_THREADS) void moddown_conv_kernel(const u64 *__restrict__ y, u64 *__restrict__ w,
                                                                  const ModConst *__restrict__ mods,
                                                                  const ModFp *__restrict__ modf,
                                                                  const u64 *__restrict__ dn_mat,
                                                                  const double *__restrict__ dn_matf, u32 level,
                                                                  u32 K, u32 L, u32 N, u32 ystride, u32 yoff, u32 kpad) {
    // kpad: special primes per row of dn_matf (K and its zero padding)
    const u32 n = blockIdx.x * KS_THREADS + threadIdx.x;
    const u32 pc = blockIdx.y;   // (item, component)
    u64 yk[KMAX];
#pragma unroll
    for (u32 k = 0; k < KMAX; ++k) {
        yk[k] = 0;
        if (k < K) yk[k] = y[((size_t)pc * ystride + yoff + k) * N + n];
    }
    const u32 i0 = blockIdx.z * DN_CHUNK, i1 = min(i0 + DN_CHUNK, level);
    if (FP) {
        // Every target below 2^50 and every special prime below 2^60 (the launcher checks): each y_k is cut into
        // three 20-bit pieces and each factor (times 2^0, 2^20, 2^40, reduced) into two 25-bit halves, all held
        // as doubles.  The 45-bit products are summed exactly by FMAs into a low and a high sum (3*KMAX terms
        // each, below 2^53), and the result is (high * 2^25 + low) mod q: the 32-bit integer multiplier, four
        // times slower per product, stays out of it.
        double yp[KMAX][3];
#pragma unroll
        for (u32 k = 0; k < KMAX; ++k) {
            const u64 v = yk[k];
            yp[k][0] = __longlong_as_double((long long)(0x4330000000000000ull | (v & 0xFFFFFu))) - 4503599627370496.0;
            yp[k][1] =
                __longlong_as_double((long long)(0x4330000000000000ull | ((v >> 20) & 0xFFFFFu))) - 4503599627370496.0;
            yp[k][2] = __longlong_as_double((long long)(0x4330000000000000ull | (v >> 40))) - 4503599627370496.0;
        }
        for (u32 i = i0; i < i1; ++i) {
            const double q = modf[i].q, u = modf[i].u;
            const double *f = dn_matf + (size_t)i * kpad * 6;
            double lo = 0.0, hi = 0.0;
#pragma unroll
            for (u32 k = 0; k < KMAX; ++k)
                if (k < K) {
#pragma unroll
                    for (u32 a = 0; a < 3; ++a) {
                        lo = fma(yp[k][a], f[(k * 3 + a) * 2 + 0], lo);
                        hi = fma(yp[k][a], f[(k * 3 + a) * 2 + 1], hi);
                    }
                }
            const double t = hi * 33554432.0;                       // exact: a power of two
            double v = fma(-rint(t * u), q, t) + lo;                // |.| < 0.75 q, plus low < 2^51
            v = fma(-rint(v * u), q, v);
            if (v < 0) v += q;
            w[((size_t)pc * level + i) * N + n] = (u64)v;
        }
    } else {
        for (u32 i = i0; i < i1; ++i) {
            u128 acc = {0, 0};
#pragma unroll
            for (u32 k = 0; k < KMAX; ++k)
                if (k < K) mac(acc, yk[k], dn_mat[(size_t)k * L + i]);
            w[((size_t)pc * level + i) * N + n] = redc_wide(acc, mods[i]);   // up to 16 products below 2^62 * q each
        }
    }
}

// ModDown between the two tile passes at N = 2^(12+LOGR), one kernel instead of three.  The last LOGR stages of the
// inverse transform of the special limbs, the base conversion P -> q_i and the first LOGR stages of the forward transform
// of the correction w all work on columns (residues 4096 apart), so a workgroup that owns a tile of 1024 coefficients
// (1024 >> LOGR columns) can do all three without leaving the CU:
//   1. wavefront k: the columns of special limb k in registers, last inverse round (which folds in
//      N^-1 (P/p_k)^-1) -> y_k in LDS;
//   2. every thread: its two coefficients' y_k cut into 30-bit pieces, then for each group of
//      MID_TG target limbs the exact sums of mid_convert -> w in LDS;
//   3. wavefront t: the columns of w_t from LDS, first forward round, out.
// At N = 2^12 (LOGR = 0) the tile passes are whole transforms and this is the conversion alone, without LDS.
// y: rows (pc*ystride + yoff + k) hold the special limbs after the inverse tile pass; w [pc][level][N] receives the
// correction ready for the forward tile pass.  Needs K <= 8, every target below 2^50 and every special prime below
// 2^60 (the launcher checks).  grid: x = column tile, y = pc.
constexpr u32 MID_TG = 8, MID_MAX_LEVEL = 32;
// KM: K rounded up to a power of two; the factor table is padded with zeros to it, so the loop has no per-prime checks
// and a target's 4 KM factors arrive through the scalar cache in one burst (with the checks the wave waited for each
// prime's six in turn).  Staging the factors in LDS instead was measured slower: broadcast reads still take an LDS issue
// slot per pair of multiply-adds.
// RESC: ModDown and rescale in one (the merged giant step's last act).  The rescale needs the dropped limb of the
// brought-down ciphertext in the coefficient domain, r = INTT(z + u P^-1)[l-1] - w_{l-1} P^-1, with z the part of the
// ciphertext that needs no ModDown; t_rows holds INTT(z + u P^-1)[l-1] and w_{l-1} is computed here first.  With
// r' = r + floor(q_{l-1}/2) mod q_{l-1}, the correction of limb i < l-1 becomes w_i P^-1 + (r' mod q_i - floor(q_{l-1}/2)
// mod q_i): one forward transform per limb serves both the ModDown and the rescale, and the rows written are those of
// the l-1 remaining limbs.  Exact modular arithmetic throughout: the same residues as ModDown followed by rescale.
template <u32 LOGR, u32 KM, bool RESC>
__global__ __launch_bounds__(MidTile<LOGR>::THREADS, 4) void moddown_mid_kernel(const u64 *__restrict__ y, u64 *__restrict__ w,
                                                          const ModConst *__restrict__ mods,
                                                          const ModFp *__restrict__ modf,
                                                          const ModFp *__restrict__ modf_dn,
                                                          const u64 *__restrict__ tw_inv,
                                                          const double *__restrict__ twf_inv,
                                                          const u64 *__restrict__ ninv_dn,
                                                          const double *__restrict__ twf_fwd,
                                                          const u32 *__restrict__ dn_mats, u32 level, u32 K, u32 L,
                                                          u32 ystride, u32 yoff, const u64 *__restrict__ t_rows,
                                                          u32 tsplit, u32 tg, bool streamed) {
    typedef MidTile<LOGR> MT;
    constexpr u32 logN = 12 + LOGR, N = 1u << logN, R = 1u << LOGR, MID_TILE = MT::SIZE, COLS = MT::COLS, PER = MT::PER;
    static_assert(MID_TG == 8 && KM <= 8, "the correction tiles reuse the 8 rows of special-limb tiles");
    __shared__ u64 ylds[LOGR ? 8 * MID_TILE : 1];
    u64 *wlds = ylds;               // y lives in registers once step 2 has read it: the same 64 KiB
    const u32 tid = threadIdx.x, lane = tid & 63, grp = __builtin_amdgcn_readfirstlane(tid / 64);   // grp < 8
    // tsplit > 1 (few polynomials): the groups of targets go to tsplit workgroups, each of which redoes step 1
    const u32 c0 = blockIdx.x % (N / MID_TILE) * COLS, tpart = blockIdx.x / (N / MID_TILE);
    const u32 pc = blockIdx.y;
    u64 yraw[2][KM];
    if constexpr (LOGR == 0) {
#pragma unroll
        for (u32 k = 0; k < KM; ++k)
#pragma unroll
            for (u32 e = 0; e < 2; ++e)                              // the tile pass was the whole transform, scaled
                yraw[e][k] = k < K ? y[((size_t)pc * ystride + yoff + k) * N + c0 + e * MT::THREADS + tid] : 0;
    } else if (grp < K) {
        const u32 gl = L + grp;
        const RowBuf src(y + ((size_t)pc * ystride + yoff + grp) * N, N);
        // the kind of the row chosen once, so that the loads of all its columns are on their way together: chosen per column, each
        // waits for the one before (a lone switch at 2^13, eight columns a thread: 7.2 us, 5.2 so; 64 of 8 special limbs 14.3 and 14.9)
        with_field(modf_dn[gl], mods, tw_inv, twf_inv, ninv_dn, gl, logN, [&](const auto &f) {
#pragma unroll
            for (u32 c = 0; c < PER; ++c) {
                const u32 col = lane + 64 * c;
                auto load = [&](u32 at, u32) { return src.load(at + c0, col); };
                auto store = [&](u32 at, u32, u64 v) { ylds[grp * MID_TILE + (at >> 12) * COLS + col] = v; };
                pass_a_body<true, LOGR>(f, c0 + col, load, store);
            }
        });
    }
    if constexpr (LOGR != 0) {
        __syncthreads();
        // the two coefficients of this thread leave LDS as they are
#pragma unroll
        for (u32 e = 0; e < 2; ++e)
#pragma unroll
            for (u32 k = 0; k < KM; ++k) yraw[e][k] = k < K ? ylds[k * MID_TILE + e * MT::THREADS + tid] : 0;
        __syncthreads();            // every thread has its y: the tile may be overwritten
    }
    u32 yp[2][KM][2];
#pragma unroll
    for (u32 e = 0; e < 2; ++e) mid_pieces<KM, 30>(yraw[e], yp[e]);
    // rescale: the dropped limb first
    double rp[2] = {0.0, 0.0}, hq = 0.0;
    const u32 n_out = RESC ? level - 1 : level;
    if (RESC) {
        const u32 il = level - 1;
        const ModFp ml = modf[il];
        FieldFp fl;
        fl.q = ml.q;
        fl.u = ml.u;
        fl.n0 = fl.n1 = 0.0;
        fl.tw = nullptr;
        hq = (double)(mods[il].q >> 1);
#pragma unroll
        for (u32 e = 0; e < 2; ++e) {
            const double wl = mid_convert<KM>(yp[e], dn_mats + (size_t)il * (KM * 4), ml.q, ml.u);
            const u32 el = e * MT::THREADS + tid;
            const double t = fl.in(t_rows[(size_t)pc * N + el / COLS * 4096 + c0 + el % COLS]);
            double r = t - wl;
            fl.norm(r);
            if (r < 0) r += ml.q;                                   // r in [0, q_last)
            r += hq;
            rp[e] = r >= ml.q ? r - ml.q : r;                       // r' = (r + h) mod q_last
        }
    }
    for (u32 i0 = tpart * tg; i0 < n_out; i0 += tsplit * tg) {
        const u32 here = min(tg, n_out - i0);
        for (u32 t = 0; t < MID_TG && t < here; ++t) {
            const u32 i = i0 + t;
            const double q = modf[i].q, u = modf[i].u;
#pragma unroll
            for (u32 e = 0; e < 2; ++e) {
                double v = mid_convert<KM>(yp[e], dn_mats + (size_t)i * (KM * 4), q, u);
                if (RESC) {
                    FieldFp fi;
                    fi.q = q;
                    fi.u = u;
                    fi.n0 = fi.n1 = 0.0;
                    fi.tw = nullptr;
                    double hi_ = hq, ri = rp[e];
                    fi.norm(hi_);                                   // floor(q_last / 2) mod q_i
                    fi.norm(ri);                                    // r' mod q_i
                    v += ri - hi_;                                  // |.| < 2q + 2^32: the forward round normalises
                }
                if constexpr (LOGR == 0)
                    w[((size_t)pc * level + i) * N + c0 + e * MT::THREADS + tid] = make_field_fp(modf[i], twf_fwd, i, logN).out(v);
                else
                    wlds[t * MID_TILE + e * MT::THREADS + tid] = (u64)__double_as_longlong(v);
            }
        }
        if constexpr (LOGR != 0) {
            __syncthreads();
            if (grp < here) {
                const u32 i = i0 + grp;
                const FieldFp ff = make_field_fp(modf[i], twf_fwd, i, logN);
                const RowBuf dst(w + ((size_t)pc * level + i) * N, N);
#pragma unroll
                for (u32 c = 0; c < PER; ++c) {
                    const u32 col = lane + 64 * c;
                    double v[R];
#pragma unroll
                    for (u32 j = 0; j < R; ++j)
                        v[j] = __longlong_as_double((long long)wlds[grp * MID_TILE + j * COLS + col]);
                    radix_fwd<LOGR>(ff, v, 0, 0);
                    // w of a large batch goes past the caches: it is read once, by the next kernel, which then finds the digit
                    // rows there (passb_final_kernel of 24 switches 524 -> 510 us)
                    if (streamed) {
#pragma unroll
                        for (u32 j = 0; j < R; ++j) dst.store<true>(j * 4096 + c0, col, ff.half(v[j]));
                    } else {
#pragma unroll
                        for (u32 j = 0; j < R; ++j) dst.store(j * 4096 + c0, col, ff.half(v[j]));
                    }
                }
            }
            __syncthreads();
        }
    }
}

// t[pc][k] = z[pc][l-1][k] + u[pc][l-1][k] P^-1 mod q_{l-1} (NTT domain; component 0: + bias[r][l-1][k], where there is one): the
// dropped limb of the ciphertext before its special-limb correction.  z_r: component-major ciphertexts [2][level][N]; u [n][2][level+K][N].
__global__ __launch_bounds__(KS_THREADS) void rescale_last_row_kernel(PtrPack z, const u64 *__restrict__ u,
                                                                      const u64 *__restrict__ bias,
                                                                      u64 *__restrict__ t,
                                                                      const ModConst *__restrict__ mods,
                                                                      u32 level, u32 K, u32 N) {
    const u32 k = blockIdx.x * KS_THREADS + threadIdx.x;
    const u32 pc = blockIdx.y, r = pc >> 1, comp = pc & 1, i = level - 1;
    const ModConst m = mods[i];
    const u64 zz = z.p[r][((size_t)comp * level + i) * N + k];
    const u64 uu = u[((size_t)pc * (level + K) + i) * N + k];
    u64 v = add_mod(zz, uu, m.q);
    if (bias && comp == 0) v = add_mod(v, bias[((size_t)r * level + i) * N + k], m.q);
    t[(size_t)pc * N + k] = v;
}

// The end of a ModDown: the forward tile pass of the correction w and what is done with it, limb i of component comp of
// ciphertext r:
//   out = z + u P^-1 - NTT(w),                                       or with RESC, on the l-1 remaining limbs,
//   out = (z + u P^-1 - NTT(w') (+ bias, component 0)) q_{l-1}^-1.
// z: ciphertexts [2][level][N], which out may be (not RESC).  Bound by memory, 32 bytes a residue at a copy's rate; as a tile
// pass and a kernel behind it, 48: nine blocks of 24 limbs at 2^16 249 -> 189 us.  grid: x = 4096-residue tiles, y = limb, z = pc
template <u32 RL, bool RESC>
__global__ __launch_bounds__(Tile<RL>::THREADS) void moddown_tile_kernel(PtrPack z, PtrPack out, const u64 *__restrict__ u,
                                                                   const u64 *__restrict__ w, const u64 *__restrict__ bias,
                                                                   const ModFp *__restrict__ modf,
                                                                   const ModConst *__restrict__ mods,
                                                                   const double *__restrict__ twf_fwd,
                                                                   const u64 *__restrict__ qlinv, u32 level, u32 K,
                                                                   u32 logN) {
    typedef Tile<RL> TL;
    __shared__ u64 lds[TL::WORDS];
    const u32 i = blockIdx.y, pc = blockIdx.z, r = pc >> 1, comp = pc & 1, tid = threadIdx.x, base = blockIdx.x << 12;
    const u64 *zr = z.p[r] + (((size_t)comp * level + i) << logN) + base;
    const u64 *ur = u + (((size_t)pc * (level + K) + i) << logN) + base;
    const u64 *br = RESC && bias && comp == 0 ? bias + (((size_t)r * level + i) << logN) + base : nullptr;
    const u64 *wr = w + (((size_t)pc * level + i) << logN);
    u64 *dst = const_cast<u64 *>(out.p[r]) + (((size_t)comp * (RESC ? level - 1 : level) + i) << logN) + base;
    const FieldFp f = make_field_fp(modf[i], twf_fwd, i, logN);
    const double c = RESC ? canonical_double(mont_mul(qlinv[i], 1, mods[i])) : 0.0;     // q_l^-1 (stored in Montgomery form)
    constexpr u32 EPP = RL < 4 ? TL::R / 2 : EPI / 2;
    pair_t zv[EPP], uv[EPP], bv[EPP];
    auto load_operands = [&](u32 i0) {
#pragma unroll
        for (u32 e = 0; e < EPP; ++e) {
            const u32 loc = TL::pair(tid, i0 + e);
            zv[e] = *reinterpret_cast<const pair_t *>(zr + loc);
            uv[e] = *reinterpret_cast<const pair_t *>(ur + loc);
            bv[e] = br ? *reinterpret_cast<const pair_t *>(br + loc) : pair_t{0, 0};
        }
    };
    if (RL < 4) load_operands(0);
    pass_b_fwd_to_lds<true, RL>(f, logN, lds, [&](u32 idx) { return wr[idx]; });
    for (u32 i0 = 0; i0 < TL::R / 2; i0 += EPP) {
        if (RL == 4) load_operands(i0);
#pragma unroll
        for (u32 e = 0; e < EPP; ++e) {
            const u32 loc = TL::pair(tid, i0 + e);
            pair_t o;
#pragma unroll
            for (u32 s = 0; s < 2; ++s) {
                const double x = (canonical_double(zv[e][s]) + canonical_double(uv[e][s])) + canonical_double(bv[e][s]) -
                                 __longlong_as_double((long long)lds[TL::slot(loc + s)]);
                o[s] = f.out(RESC ? f.mul(x, c) : x);
            }
            *reinterpret_cast<pair_t *>(dst + loc) = o;
        }
    }
}

// Whether the fused kernel applies to this parameter set at this level.
bool moddown_mid_ok(const ckks_params *p, u32 level) {
    bool ok = p->logN >= 12 && p->logN <= 16 && p->dn_fp && p->K >= 1 && p->K <= 8 && level <= MID_MAX_LEVEL;
    for (u32 i = 0; i < level; ++i) ok = ok && (p->mod[i] >> 50) == 0;
    return ok;
}

typedef decltype(&moddown_mid_kernel<4, 8, false>) moddown_mid_t;
template <u32 LOGR, bool RESC>
static moddown_mid_t moddown_mid_for(u32 km) {
    return km == 1 ? moddown_mid_kernel<LOGR, 1, RESC> : km == 2 ? moddown_mid_kernel<LOGR, 2, RESC>
         : km == 4 ? moddown_mid_kernel<LOGR, 4, RESC> : moddown_mid_kernel<LOGR, 8, RESC>;
}
template <bool RESC>
static moddown_mid_t moddown_mid_for(const ckks_params *p) {
    const u32 km = pad_pow2(p->K);
    switch (p->logN) {
        case 12: return moddown_mid_for<0, RESC>(km);
        case 13: return moddown_mid_for<1, RESC>(km);
        case 14: return moddown_mid_for<2, RESC>(km);
        case 15: return moddown_mid_for<3, RESC>(km);
        default: return moddown_mid_for<4, RESC>(km);
    }
}

// Targets of a group: as few groups as there can be, of one size (a lone call waits for the longest: ModDown of 17 limbs, 8 + 8 + 1 /
// 6 + 6 + 5 targets: 21.1 / 19.1 us; ModUp, whose last digit has 24 targets there, gains nothing by it), and where these leave
// CUs without a workgroup, as many as there are CUs: small groups convert less behind one another.  us, groups as few as there can be /
// up to 256 workgroups in both conversions: one rotation at 2^16, 12 + 6 primes of 40 and 49 bits, level 6, one digit 55.5 and 48.9;
// 24 + 8 primes, level 1 / 4 / 6 53.6 / 57.5 / 60.6 and 48.8 / 50.0 / 52.6; 2^15, 8 + 4, one digit of four 51.7 and 46.4; 2^14, 6 + 2
// 47.8 and 44.3; 2^13, 8 + 8 52.3 and 45.2.  Up to 512, ModDown at 2^16 takes 3 % more than with as few as there can be.
static u32 group_size(u32 workgroups, u32 targets) {
    const u32 groups = std::max<u32>({1, (targets + MID_TG - 1) / MID_TG, std::min(targets, 256 / workgroups)});
    return std::max<u32>(1, (targets + groups - 1) / groups);
}

// Workgroups among which ModDown splits the target groups of a tile: up to three for each of the 256 CUs, which run two at a
// time.  The line hardly matters: whole calls with at most 256 / 384 / 512 / 768 / 1024 / 1536 workgroups, us: one rotation at
// 2^16, level 24 134.4 / 133.3 / 133.4 / 133.2 / 133.5 / 133.3, three at level 17 189.7 / 189.6 / 189.5 / 186.4 / 186.5 / 190.4,
// two at level 24 185.5 / 185.4 / 186.7 / 184.5 / 184.5 / 184.8; products, and calls of 2^15 and less, within 0.5 %.
static u32 target_split(u32 workgroups, u32 groups) { return std::max<u32>(1, std::min<u32>(groups, 768 / workgroups)); }

static void launch_moddown_mid(const ckks_params *p, const u64 *y, u64 *w, u32 n, u32 level, u32 ystride, u32 yoff,
                               hipStream_t stream, const u64 *t_rows = nullptr) {
    const u32 tiles = p->N / mid_tile(p), threads = mid_tile(p) / 2;
    const u32 n_out = level - (t_rows ? 1 : 0), wgs = tiles * n * 2, tg = group_size(wgs, n_out);
    const u32 tsplit = target_split(wgs, (n_out + tg - 1) / tg);
    hipLaunchKernelGGL(t_rows ? moddown_mid_for<true>(p) : moddown_mid_for<false>(p), dim3(tiles * tsplit, n * 2),
                       dim3(threads), 0, stream, y, w, p->d_mod, p->d_modf, p->d_modf_dn, p->d_tws_inv, p->d_twf_inv,
                       p->d_ninvs_dn, p->d_twf_fwd, p->d_dn_mats, level, p->K, p->L, ystride, yoff, t_rows, tsplit, tg,
                       (size_t)n * 2 * level * p->N * sizeof(u64) > STREAM_BYTES);
}

// base conversion P -> q_i of n*2 polynomials; the rows of polynomial pc start at row pc * ystride + yoff of y
static void launch_moddown_conv(const ckks_params *p, const u64 *y, u64 *w, u32 n, u32 level, u32 ystride, u32 yoff,
                                hipStream_t stream) {
    const dim3 grid(p->N / KS_THREADS, n * 2, (level + DN_CHUNK - 1) / DN_CHUNK);
    bool fp = p->dn_fp;        // fp64 sums need every target below 2^50 and every special prime below 2^60
    for (u32 i = 0; i < level; ++i) fp = fp && (p->mod[i] >> 50) == 0;
#define CONV_LAUNCH(KM, FPK)                                                                                      \
    hipLaunchKernelGGL((moddown_conv_kernel<KM, FPK>), grid, dim3(KS_THREADS), 0, stream, y, w, p->d_mod, p->d_modf, \
                       p->d_dn_mat, p->d_dn_matf, level, p->K, p->L, p->N, ystride, yoff, pad_pow2(p->K))
    if (p->K <= 8) {
        if (fp) CONV_LAUNCH(8, true); else CONV_LAUNCH(8, false);
    } else {
        if (fp) CONV_LAUNCH(MAX_DIGIT, true); else CONV_LAUNCH(MAX_DIGIT, false);
    }
#undef CONV_LAUNCH
}

// dst[comp][i][k] (+)= (u_{q_i} - NTT(w_i)) * P^-1  (+ sigma_g(c0)[i][k] for comp 0)
__global__ __launch_bounds__(KS_THREADS) void moddown_final_kernel(ItemPack pack, const u64 *__restrict__ u,
                                                                   const u64 *__restrict__ w,
                                                                   const ModConst *__restrict__ mods, u32 level, u32 K,
                                                                   u32 logN) {
    const u32 N = 1u << logN;
    const u32 k = blockIdx.x * KS_THREADS + threadIdx.x;
    const u32 i = blockIdx.y, r = blockIdx.z >> 1, comp = blockIdx.z & 1;
    const u32 Wl = level + K;
    const SwitchItem &it = pack.it[r];
    const ModConst m = mods[i];
    const u64 uq = u[(((size_t)r * 2 + comp) * Wl + i) * N + k];
    const u64 wq = w[(((size_t)r * 2 + comp) * level + i) * N + k];
    u64 v = sub_mod(uq, wq, m.q);
    if (comp == 0 && it.c0) v = add_mod(v, it.c0[(size_t)i * N + galois_index(k, (u32)it.galois_elt, logN)], m.q);
    u64 *dst = it.dst + ((size_t)comp * level + i) * N + k;
    if (it.add) v = add_mod(v, it.add[((size_t)comp * level + i) * N + k], m.q);
    if (it.balanced && (m.q >> 50) == 0) v = balanced_bits(v, m.q);
    *dst = v;
}

// ---- kernels fused into the tile passes, N = 2^12 .. 2^17 ------------------------------------------
// Key inner product on the special limbs feeding straight into the first pass of their inverse transform:
// row (comp, k, r) of y = INTT-pass-B( sum_j sigma_g(d_j)[p_k] * key_j[comp][p_k] ).
// grid: x = tile of 4096, y = ((k*n + r)*2 + comp): the two components of an item (same digit reads) and the
// items of a batch that share a key sit next to each other and, with 16 tiles per row, on the same XCD.
// KEY_NT: key rows are read with non-temporal loads.  Right when every item has a key of its own (the rows are used
// once and would only push the digit rows, which every item re-reads, out of L2); wrong when neighbouring items share
// a key, where it is the cached line that lets the second and third reader skip HBM.
template <bool NT>
__device__ __forceinline__ pair_t load_key(const pair_t *p) {
    return NT ? __builtin_nontemporal_load(p) : *p;
}

template <bool KEY_NT, bool PAIR, u32 RL>
__global__ __launch_bounds__(Tile<RL>::THREADS) void ip_intt_kernel(ItemPack pack, u64 *__restrict__ y,
                                                              const ModConst *__restrict__ mods,
                                                              const ModFp *__restrict__ modf,
                                                              const u64 *__restrict__ tw_inv,
                                                              const double *__restrict__ twf_inv,
                                                              const u64 *__restrict__ ninv, u32 n, u32 level, u32 K,
                                                              u32 L, u32 beta, u32 logN) {
    typedef Tile<RL> TL;
    __shared__ u64 lds[TL::WORDS];
    const u32 N = 1u << logN;
    const u32 comp = blockIdx.y & 1, k = uniform_div(blockIdx.y >> 1, n), r = (blockIdx.y >> 1) - k * n;
    const u32 gl = L + k, t = level + k, Wl = level + K, Wt = L + K;
    const SwitchItem &it = pack.it[r];
    const ModConst m = mods[gl];
    const u64 *dig = it.digits + (size_t)t * N;
    const u64 *key = it.key + ((size_t)comp * Wt + gl) * N;
    const u32 g = (u32)it.galois_elt;
    u64 *out = y + (((size_t)r * 2 + comp) * K + k) * N;
    auto store = [&](u32 idx, u64 v) { out[idx] = v; };
    // inner product into LDS on pairs of adjacent residues (16-byte key loads), two pairs (RL < 4: all of them) at a time so
    // that their loads are in flight together
    const u32 tid = threadIdx.x, base = blockIdx.x << 12;
    constexpr u32 EPP = RL < 4 ? TL::R / 2 : EPI / 2;
    for (u32 i0 = 0; i0 < TL::R / 2; i0 += EPP) {
        pair_t dv[EPP][MAX_BETA], kv[EPP][MAX_BETA];
        u32 kp[EPP];
#pragma unroll
        for (u32 e = 0; e < EPP; ++e) {
            const u32 idx = base + TL::pair(tid, i0 + e);
            kp[e] = galois_index(idx, g, logN);
#pragma unroll
            for (u32 j = 0; j < MAX_BETA; ++j)
                if (j < beta) {
                    dv[e][j] = load_two<PAIR>(dig + (size_t)j * Wl * N, kp[e]);
                    kv[e][j] = load_key<KEY_NT>(reinterpret_cast<const pair_t *>(key + (size_t)j * 2 * Wt * N + idx));
                }
        }
#pragma unroll
        for (u32 e = 0; e < EPP; ++e) {
            const u32 loc = TL::pair(tid, i0 + e);
#pragma unroll
            for (u32 j = 0; j < MAX_BETA; ++j)
                if (j < beta) dv[e][j] = turned<PAIR>(dv[e][j], kp[e]);
#pragma unroll
            for (u32 z = 0; z < 2; ++z) {
                u128 acc = {0, 0};
#pragma unroll
                for (u32 j = 0; j < MAX_BETA; ++j)
                    if (j < beta) mac(acc, dv[e][j][z], kv[e][j][z]);
                // up to four products of residues below 2^62: a sum below q 2^64 (redc_wide's loop is a branch per residue: 24
                // switches at 2^14 30.4 us, without it 26.3, one at 2^16 18.7 and 16.2, 27 346 and 340)
                static_assert(MAX_BETA <= 4, "the sum has to stay below q 2^64");
                lds[TL::slot(loc + z)] = redc(acc, m);
            }
        }
    }
    with_field(modf[gl], mods, tw_inv, twf_inv, ninv, gl, logN,
               [&](const auto &f) { pass_b_inv_from_lds<RL>(f, logN, lds, store); });
}

// Last pass of the forward transform of w fused with the rest of the key switch on limb q_i:
//   dst[comp][i] (+)= sum_j sigma_g(d_j)[q_i] * key_j[comp][q_i] - NTT(w)[i]  (+ sigma_g(c0)[i] if comp = 0)
// (the keys and w carry the P^-1 of ModDown).
// grid: x = tile of 4096, y = ((i*n + r)*2 + comp), neighbours share digit and key lines in L2 as above.
// CONV (N = 2^12): w holds the K special rows of an (item, component) instead, scaled by (P/p_k)^-1, and the workgroup converts
// its row of the correction from them itself (dn_mats: the factors, kpad source rows a target).
template <bool KEY_NT, bool PAIR, u32 RL, bool CONV>
__global__ __launch_bounds__(Tile<RL>::THREADS) void passb_final_kernel(ItemPack pack, const u64 *__restrict__ w,
                                                                  const u32 *__restrict__ dn_mats, u32 kpad,
                                                                  const ModConst *__restrict__ mods,
                                                                  const ModFp *__restrict__ modf,
                                                                  const u64 *__restrict__ tw_fwd,
                                                                  const double *__restrict__ twf_fwd,
                                                                  const u64 *__restrict__ ninv, u32 n, u32 level,
                                                                  u32 K, u32 L, u32 beta, u32 alpha, u32 logN) {
    typedef Tile<RL> TL;
    static_assert(RL == 4 || !PAIR, "operands that share a register with gathered ones are not turned");
    __shared__ u64 lds[TL::WORDS];
    const u32 N = 1u << logN;
    const u32 comp = blockIdx.y & 1, i = uniform_div(blockIdx.y >> 1, n), r = (blockIdx.y >> 1) - i * n;
    const u32 Wl = level + K, Wt = L + K;
    const SwitchItem &it = pack.it[r];
    const ModConst m = mods[i];
    const u64 *wrow = w + (((size_t)r * 2 + comp) * level + i) * N;
    // row of limb i in digit j; the digit that owns limb i is not stored: its row is the source's own
    const u64 *drow[MAX_BETA];
    const u32 own = uniform_div(i, alpha);
#pragma unroll
    for (u32 j = 0; j < MAX_BETA; ++j)
        drow[j] = j == own ? it.c1 + (size_t)i * N : it.digits + ((size_t)j * Wl + i) * N;
    const u64 *key = it.key + ((size_t)comp * Wt + i) * N;
    const u64 *c0 = it.c0 + (size_t)i * N;
    u64 *dst = it.dst + ((size_t)comp * level + i) * N;
    const u32 g = (u32)it.galois_elt;
    const bool accumulate = it.add != nullptr;
    const u64 *add = it.add + ((size_t)comp * level + i) * N + (blockIdx.x << 12);   // read only if it.add is there
    auto load = [&](u32 idx) -> u64 { return __builtin_nontemporal_load(wrow + idx); };
    const ModFp mf = modf[i];
    // epilogue on pairs of adjacent residues (16-byte accesses to the streamed operands), two pairs at a time so
    // that their loads are in flight together (RL < 4: all of them, during the transform).  Keys, w and the output are streamed
    // once: non-temporal, so that they do not push the digit rows (re-read by every item of the batch) out of L2.
    const u32 tid = threadIdx.x, base = blockIdx.x << 12;
    constexpr u32 EPP = RL < 4 ? TL::R / 2 : EPI / 2;
    const bool fold = comp == 0 && it.c0;
    pair_t dv[EPP][MAX_BETA], kv[EPP][MAX_BETA], cv[EPP], ov[EPP];
    u32 kp[EPP];
    auto load_add = [&](u32 loc) { return __builtin_nontemporal_load(reinterpret_cast<const pair_t *>(add + loc)); };
    auto load_operands = [&](u32 i0) {
#pragma unroll
        for (u32 e = 0; e < EPP; ++e) {
            const u32 idx = base + TL::pair(tid, i0 + e);
            kp[e] = galois_index(idx, g, logN);
#pragma unroll
            for (u32 j = 0; j < MAX_BETA; ++j)
                if (j < beta) {
                    dv[e][j] = load_two<PAIR>(drow[j], kp[e]);
                    kv[e][j] = load_key<KEY_NT>(reinterpret_cast<const pair_t *>(key + (size_t)j * 2 * Wt * N + idx));
                }
            cv[e] = fold ? load_two<PAIR>(c0, kp[e]) : accumulate && RL < 4 ? load_add(TL::pair(tid, i0 + e)) : pair_t{0, 0};
            if (RL == 4) ov[e] = accumulate ? load_add(TL::pair(tid, i0 + e)) : pair_t{0, 0};
        }
    };
    if (CONV) {
        u64 raw[TL::R];
        tile_convert<RL, 30>(w + ((size_t)r * 2 + comp) * K * 4096, K, dn_mats + (size_t)i * (kpad * 4),
                             [&](u32 j, u64 s0, u64 s1) { raw[j] = (u64)__double_as_longlong(mid_reduce(s0, s1, mf.q, mf.u)); });
        if (RL < 4) load_operands(0);
        pass_b_fwd_from_regs<true, RL, true>(make_field_fp(mf, twf_fwd, i, 12), 12, lds, raw, 0);
    } else if (mf.ok) {   // the fp64 epilogue takes the transformed correction as doubles, |x| <= q/2
        if (RL < 4) load_operands(0);
        pass_b_fwd_to_lds<true, RL>(make_field_fp(mf, twf_fwd, i, logN), logN, lds, load);
    } else {       // the integer transforms have no registers left for them
        with_int_field(mf, mods, tw_fwd, ninv, i, logN,
                       [&](const auto &f) { pass_b_fwd_to_lds<false, RL>(f, logN, lds, load); });
        if (RL < 4) load_operands(0);
    }
    for (u32 i0 = 0; i0 < TL::R / 2; i0 += EPP) {
        if (RL == 4) load_operands(i0);
#pragma unroll
        for (u32 e = 0; e < EPP; ++e) {
            const u32 loc = TL::pair(tid, i0 + e);
            // RL < 4: one array for c0 or the addend (128 registers is what 16 wavefronts a workgroup leave); where both are
            // added, the addend comes now
            if (RL < 4) ov[e] = accumulate && fold ? load_add(loc) : pair_t{0, 0};
            __builtin_amdgcn_sched_barrier(0);
            cv[e] = turned<PAIR>(cv[e], kp[e]);
#pragma unroll
            for (u32 j = 0; j < MAX_BETA; ++j)
                if (j < beta) dv[e][j] = turned<PAIR>(dv[e][j], kp[e]);
            pair_t out;
#pragma unroll
            for (u32 z = 0; z < 2; ++z) {
                if (CONV || mf.ok) {
                    // primes below 2^50: exact fp64 sums, keys are balanced doubles
                    MacSum sum{MAC_H0, 0.0};
#pragma unroll
                    for (u32 j = 0; j < MAX_BETA; ++j)
                        if (j < beta) sum.mac(canonical_double(dv[e][j][z]), __longlong_as_double((long long)kv[e][j][z]));
                    sum.fold(mf.q, mf.u);
                    sum.l += (canonical_double(cv[e][z]) + canonical_double(ov[e][z])) -
                             __longlong_as_double((long long)lds[TL::slot(loc + z)]);
                    if (it.balanced)
                        out[z] = (u64)__double_as_longlong(fma(-rint(sum.l * mf.u), mf.q, sum.l));
                    else
                        out[z] = sum.canonical(mf.q, mf.u);
                } else {
                    u128 acc = {0, 0};
#pragma unroll
                    for (u32 j = 0; j < MAX_BETA; ++j)
                        if (j < beta) mac(acc, dv[e][j][z], kv[e][j][z]);
                    u64 v = sub_mod(redc(acc, m), lds[TL::slot(loc + z)], m.q);    // as in ip_intt_kernel
                    v = add_mod(v, cv[e][z], m.q);
                    out[z] = add_mod(v, ov[e][z], m.q);
                }
            }
            __builtin_nontemporal_store(out, reinterpret_cast<pair_t *>(dst + base + loc));
        }
    }
}

// (out0, out1, t2) = (a0*b0, a0*b1 + a1*b0, a1*b1), pointwise on limb blockIdx.y
__global__ __launch_bounds__(KS_THREADS) void tensor_kernel(const u64 *__restrict__ a, const u64 *__restrict__ b,
                                                            u64 *__restrict__ out, u64 *__restrict__ t2,
                                                            const ModConst *__restrict__ mods, u32 level, u32 N) {
    const u32 k = blockIdx.x * KS_THREADS + threadIdx.x;
    const u32 i = blockIdx.y;
    const ModConst m = mods[i];
    const size_t o0 = (size_t)i * N + k, o1 = ((size_t)level + i) * N + k;
    const u64 a0 = a[o0], a1 = a[o1];
    const u64 b0 = mont_mul(b[o0], m.r2, m), b1 = mont_mul(b[o1], m.r2, m);   // Montgomery form
    out[o0] = mont_mul(a0, b0, m);
    out[o1] = add_mod(mont_mul(a0, b1, m), mont_mul(a1, b0, m), m.q);
    t2[o0] = mont_mul(a1, b1, m);
}

size_t digits_words(const ckks_params *p, u32 level) {
    u32 beta = (level + p->alpha - 1) / p->alpha;
    return (size_t)beta * (level + p->K) * p->N;
}

size_t switch_scratch_words(const ckks_params *p, u32 level, u32 n_items) {
    return (size_t)n_items * 2 * ((size_t)(level + p->K) + level) * p->N;
}

// forward transform (the passes of pass_mask) of the converted rows; the digit's own limbs are not filled and skipped
static int transform_digits(ckks_params *p, u32 level, u32 n, u64 *d_digits, hipStream_t stream, u32 pass_mask) {
    const u32 Wl = level + p->K, alpha = p->alpha, beta = (level + alpha - 1) / alpha;
    LimbIds ids;
    auto row_id = [&](u32 j, u32 t) -> uint8_t {
        const u32 lo = j * alpha, hi = std::min(lo + alpha, level);
        if (t >= lo && t < hi) return (uint8_t)SKIP_ROW;
        return (uint8_t)(t < level ? t : p->L + (t - level));
    };
    if (beta * Wl <= MAX_ROW_IDS) {
        for (u32 j = 0; j < beta; ++j)
            for (u32 t = 0; t < Wl; ++t) ids.id[j * Wl + t] = row_id(j, t);
        return launch_ntt(p, d_digits, ids, beta * Wl, n * beta * Wl, false, stream, pass_mask);
    }
    for (u32 r = 0; r < n; ++r)
        for (u32 j = 0; j < beta; ++j) {
            for (u32 t = 0; t < Wl; ++t) ids.id[t] = row_id(j, t);
            const int rc = launch_ntt(p, d_digits + ((size_t)r * beta + j) * Wl * p->N, ids, Wl, Wl, false, stream, pass_mask);
            if (rc) return rc;
        }
    return CKKS_OK;
}

// the kernels that convert between the column passes (or, at N = 2^12, in the transforms) apply to ModUp
static bool modup_mid_ok(const ckks_params *p, u32 level) {
    bool ok = p->logN >= 12 && p->logN <= 16 && p->alpha <= 8 && p->K <= 8;
    for (u32 i = 0; i < level; ++i) ok = ok && (p->mod[i] >> 50) == 0;
    for (u32 k = 0; k < p->K; ++k) ok = ok && (p->mod[p->L + k] >> 60) == 0;
    return ok;
}
// constants of the first pass of the decomposition's inverse transform: at N = 2^12 it is the whole one and scales for ModUp
static const ModFp *decompose_modf(const ckks_params *p, const LevelTables *lt) {
    return p->logN == 12 && modup_mid_ok(p, lt->level) ? lt->d_modf_up : p->d_modf;
}

static int decompose_from_tmp(ckks_params *p, const LevelTables *lt, u32 n, u64 *d_digits, u64 *d_tmp, hipStream_t stream,
                              bool half);

// c1[r] [level][N] NTT domain (n <= ROT_BATCH device pointers) -> d_digits [n][beta][level+K][N] NTT domain;
// d_tmp [n][level][N] scratch.
int decompose(ckks_params *p, const u64 *const *c1, u32 n, u32 level, u64 *d_digits, u64 *d_tmp,
              hipStream_t stream, bool half) {
    if (n == 0) return CKKS_OK;
    const u32 N = p->N;
    const LevelTables *lt = nullptr;
    int rc = p->level_tables(level, &lt);
    if (rc) return rc;
    PtrPack src;
    for (u32 r = 0; r < ROT_BATCH; ++r) src.p[r] = c1[r < n ? r : 0];
    if (fast_ring(p)) {
        const bool wide = wide_tiles((u64)(N >> 12) * n * level);
        hipLaunchKernelGGL(wide ? gather_intt_kernel<WIDE_RL> : gather_intt_kernel<4>, dim3(N >> 12, n * level),
                           dim3(tile_threads(wide)), 0, stream, src, d_tmp, p->d_mod, decompose_modf(p, lt), p->d_tws_inv,
                           p->d_twf_inv, p->d_ninvs, level, p->logN);
        CKKS_LAUNCH_CHECK("gather_intt_kernel");
        p->limb_ntts += (u64)n * level;
    } else {
        LimbIds ids;
        for (u32 i = 0; i < level; ++i) ids.id[i] = (uint8_t)i;
        hipLaunchKernelGGL(gather_c1_kernel, dim3(N / KS_THREADS, level, n), dim3(KS_THREADS), 0, stream, src, d_tmp,
                           level, N);
        CKKS_LAUNCH_CHECK("gather_c1_kernel");
        rc = launch_ntt(p, d_tmp, ids, level, n * level, true, stream);
        if (rc) return rc;
    }
    return decompose_from_tmp(p, lt, n, d_digits, d_tmp, stream, half);
}

// The rest of it: d_tmp holds the polynomials after the first pass of their inverse transform (plain-kernel rings: the whole).
static int decompose_from_tmp(ckks_params *p, const LevelTables *lt, u32 n, u64 *d_digits, u64 *d_tmp, hipStream_t stream,
                              bool half) {
    const u32 N = p->N, K = p->K, L = p->L, level = lt->level, Wl = level + K, alpha = p->alpha, beta = lt->beta;
    bool all_fp = true;
    for (u32 i = 0; i < level; ++i) all_fp = all_fp && (p->mod[i] >> 50) == 0;
    if (modup_mid_ok(p, level)) {
        if (p->logN == 12 && !half) {
            const bool wide_up = wide_tiles((u64)n * beta * Wl - (u64)n * level);
            hipLaunchKernelGGL(wide_up ? modup_tile_kernel<WIDE_RL> : modup_tile_kernel<4>, dim3(Wl, beta, n),
                               dim3(tile_threads(wide_up)), 0, stream, d_tmp, d_digits, p->d_mod, p->d_modf, p->d_twf_fwd,
                               p->d_tws_fwd, p->d_ninvs, lt->d_up_ft, lt->d_up_mats, level, K, L, alpha, pad_pow2(alpha), beta);
            CKKS_LAUNCH_CHECK("modup_tile_kernel");
            p->limb_ntts += (u64)n * beta * Wl - (u64)n * level;
            return CKKS_OK;
        }
        // the column passes of both transforms ride in the base conversion: c1 read once, digits written once
        const u32 nt = Wl - std::min(alpha, level), tgroups = (nt + UP_TG - 1) / UP_TG, tiles = N / mid_tile(p), wgs = n * beta * tiles;
        // all target groups apart below 1024 workgroups (two per CU run at a time): one rotation at 2^16, level 24 / 17 / 9, two
        // at level 24, a product and rescale at 2^16 and 2^15 133.4 / 120.4 / 83.8, 184.2, 188.5 and 85.2 us; never split 135.0 /
        // 123.8 / 88.8, 186.0, 190.3 and 89.6; as many parts as make up to 256, 512, 768 or 1536 workgroups within 0.5 % of either
        const u32 tg = wgs * tgroups < 256 ? group_size(wgs, nt) : UP_TG;
        const u32 tsplit = wgs < 1024 ? (nt + tg - 1) / tg : 1;
        hipLaunchKernelGGL(modup_mid_for(p), dim3(tiles * tsplit, beta, n), dim3(mid_tile(p) / 2), 0, stream, d_tmp,
                           d_digits, p->d_mod, p->d_modf, lt->d_modf_up, p->d_twf_inv, p->d_twf_fwd, p->d_tws_fwd,
                           p->d_ninvs, lt->d_up_ft, lt->d_up_mats, level, K, L, alpha, beta, tsplit, tg);
        CKKS_LAUNCH_CHECK("modup_mid_kernel");
        p->limb_ntts += (u64)n * beta * Wl - (u64)n * level;
        return half ? CKKS_OK : transform_digits(p, level, n, d_digits, stream, 2);
    }
    if (fast_ring(p)) {
        LimbIds ids;
        for (u32 i = 0; i < level; ++i) ids.id[i] = (uint8_t)i;
        const int rc = launch_ntt(p, d_tmp, ids, level, n * level, true, stream, 2);
        if (rc) return rc;
    }
    // two launches: the ciphertext-prime targets (fp64 arithmetic when every active prime is below 2^50) and the
    // special-prime targets (integer arithmetic); each keeps only its own form of y in registers
#define MODUP_LAUNCH(A, FPK, T0, T1)                                                                               \
    hipLaunchKernelGGL((modup_kernel<A, 2, FPK>), dim3(N / KS_THREADS / 2, beta, n), dim3(KS_THREADS), 0, stream,   \
                       d_tmp, d_digits, p->d_mod, p->d_modf, lt->d_up_inv, lt->d_up_mat, lt->d_up_matf, level, K,   \
                       L, alpha, N, beta, T0, T1)
    if (alpha <= 8) {
        if (all_fp)
            MODUP_LAUNCH(8, true, 0u, level);
        else
            MODUP_LAUNCH(8, false, 0u, level);
        MODUP_LAUNCH(8, false, level, Wl);
    } else {
        if (all_fp)
            MODUP_LAUNCH(MAX_DIGIT, true, 0u, level);
        else
            MODUP_LAUNCH(MAX_DIGIT, false, 0u, level);
        MODUP_LAUNCH(MAX_DIGIT, false, level, Wl);
    }
#undef MODUP_LAUNCH
    CKKS_LAUNCH_CHECK("modup_kernel");
    return transform_digits(p, level, n, d_digits, stream, half ? 1 : 3);
}

static u32 build_pack(const SwitchItem *items, u32 n, ItemPack &pack) {
    for (u32 r = 0; r < ROT_BATCH; ++r) pack.it[r] = items[r < n ? r : 0];
    u32 n_groups = 0;
    for (u32 r = 0; r < n;) {
        u32 c = 1;
        while (r + c < n && c < KEY_GROUP && items[r + c].key == items[r].key &&
               items[r + c].galois_elt == items[r].galois_elt)
            ++c;
        pack.grp_first[n_groups] = (uint8_t)r;
        pack.grp_count[n_groups] = (uint8_t)c;
        ++n_groups;
        r += c;
    }
    for (u32 g = n_groups; g < ROT_BATCH; ++g) pack.grp_first[g] = pack.grp_count[g] = 0;
    return n_groups;
}

// A workgroup of merged_tile_kernel is a chain of all rotations and digits, so few of them leave the chip idle that long, and 512
// fit at a time.  Workgroups (ring, ciphertexts, digits), whole calls with 15 rotations, separate tile passes /
// merged_tile_kernel, us (before the folding butterflies; with them 288 and 320 of 50- and 60-bit primes, (2^14, 9, 3) 680 / 662
// and (2^14, 10, 3) 793 / 705):
//   up to three digits: 256 (2^15, 2, 3) 767 / 826, 288 (2^13, 12, 2) 675 / 656, 312 (2^15, 3, 3) 864 / 907, 320 (2^16, 1, 2)
//     851 / 821, 384 (2^15, 3, 3) 1033 / 988, 512 (2^14, 16, 3) 1606 / 1109, 544 (2^14, 17, 3) 1720 / 1171;
//   more digits, of few ciphertexts: longer chains, beside a separate kernel that reads a key once for three ciphertexts: 320
//     (2^16, 2, 4) 1074 / 1157, 336 (2^14, 4, 6) 1512 / 1564, 480 (2^16, 3, 4) 1449 / 1328; of more: 336 (2^15, 7, 5) 1426 / 1368;
//   ciphertext primes from 2^50 up: the transforms of the chain take twice as long, and a round nearly empty, of two per CU on
//     the XCD with most units, costs more than the fusion gives: 384 (2^15, 3, 3) 1619 / 1692, 440 (2^14, 22, 4; two rounds on
//     half of the XCDs) 2393 / 2612, 512 (2^15, 4, 3) 2083 / 1973, 576 (2^14, 9, 5) 3438 / 3576, 640 (2^14, 20, 3) 2728 / 2600,
//     792 (2^14, 9, 5) 4517 / 4646, 896 (2^14, 14, 5) 5211 / 5006, 1160 (2^14, 29, 4) 5510 / 5200; two digits: 352 (2^12, 32, 2)
//     1271 / 1176.
// More rows of digits than one row map describes: their own tile passes are a launch per digit and ciphertext (2^14, 11
// ciphertexts, 12 digits: 19130 / 3783).
// With ciphertext primes of 58 and 60 bits that fold (both are measured, 15 rotations, 58 / 60 bits) the line for integer rows is
// within 5 % of the faster side, on either: just below it 384 (2^15, 3, 3) 1369 / 1342 and 1310 / 1310, (2^15, 4, 3) 1358 / 1315 and 1329 /
// 1300, 400 (2^14, 10, 3) 1368 / 1314 and 1343 / 1289, 440 (2^14, 22, 4) 1943 / 2048 and 1941 / 2046, 576 (2^14, 9, 5) 2790 / 2861 and 2688 /
// 2706, (2^14, 12, 4) 2251 / 2309 and 2216 / 2288; above it 512 (2^15, 4, 3) 1803 / 1643 and 1754 / 1557, 640 (2^14, 20, 3) 2226 / 2094
// and 2219 / 2074, 896 (2^14, 14, 5) 4295 / 4008 and 4119 / 3898.
bool merged_from_half(const ckks_params *p, u32 level, u32 n) {
    const u32 Wl = level + p->K, beta = (level + p->alpha - 1) / p->alpha, units = (p->N >> 12) * Wl;
    const u32 workgroups = units * n;                            // at most 2^5 * 64 * 32
    if (!fast_ring(p) || workgroups < 320) return false;
    if (beta * Wl > MAX_ROW_IDS) return true;
    u32 n_int = 0;
    for (u32 i = 0; i < level; ++i) n_int += (p->mod[i] >> 50) != 0;
    if (2 * n_int > level && beta > 2) {
        const u32 rounds = ((units + 7) / 8 * n + 63) / 64;
        return workgroups >= (beta == 3 ? 640u : 1152u) || workgroups >= 448 * rounds;
    }
    return beta < 4 || n > 4 || workgroups >= 384;
}

// Merged giant step, part 1: d_u[r] (+)= the key inner products of rots.n_rot rotations of ciphertext r over all
// level+K limbs (NTT domain), dst_r.c0 += the rotated c0 parts.  d_u [n][2][level+K][N].
int switch_accumulate_merged(ckks_params *p, u32 level, const MergedRot &rots, u32 n, const u64 *d_digits,
                             const u64 *c0_base, size_t c0_stride_r, u64 *dst_base, size_t dst_stride, u64 *d_u,
                             bool accumulate, bool half, hipStream_t stream) {
    if (n == 0 || rots.n_rot == 0) return CKKS_OK;
    if (n > ROT_BATCH || rots.n_rot > MERGE_GROUP) {
        set_error("switch_accumulate_merged: %u ciphertexts x %u rotations exceed one launch", n, rots.n_rot);
        return CKKS_E_INVAL;
    }
    const u32 N = p->N, K = p->K, L = p->L, Wl = level + K;
    const u32 beta = (level + p->alpha - 1) / p->alpha;
    if (half) {
        LimbIds rows;                                            // the longest rows, those of larger primes, first
        u32 n_rows = 0;
        for (u32 pass = 0; pass < 2; ++pass)
            for (u32 t = Wl; t-- > 0;)
                if ((p->mod[t < level ? t : L + (t - level)] >> 50 == 0) == (pass == 1)) rows.id[n_rows++] = (uint8_t)t;
        const u32 units = ((N >> 12) * Wl + 7) / 8 * 8;
        hipLaunchKernelGGL(merged_tile_kernel<3>, dim3(units * n), dim3(Tile<3>::THREADS), 0, stream, rots, d_digits,
                           digits_words(p, level), c0_base, c0_stride_r, dst_base, dst_stride, d_u, p->d_mod, p->d_modf,
                           p->d_tws_fwd, p->d_twf_fwd, p->d_ninvs, n, level, K, L, beta, p->alpha, p->logN,
                           accumulate ? 1u : 0u, rows);
        CKKS_LAUNCH_CHECK("merged_tile_kernel");
        return CKKS_OK;
    }
    const u32 groups = (n + MR - 1) / MR;
    LimbIds fp_rows, int_rows;
    u32 n_fp = 0, n_int = 0;
    for (u32 t = 0; t < Wl; ++t)
        if (t < level && (p->mod[t] >> 50) == 0)
            fp_rows.id[n_fp++] = (uint8_t)t;
        else
            int_rows.id[n_int++] = (uint8_t)t;
    if (n_fp)
        hipLaunchKernelGGL(merged_ip_kernel<true>, dim3(N / KS_THREADS * groups, n_fp), dim3(KS_THREADS), 0, stream, rots,
                           d_digits, digits_words(p, level), c0_base, c0_stride_r, dst_base, dst_stride, d_u, p->d_mod, n,
                           level, K, L, beta, p->alpha, p->logN, accumulate ? 1u : 0u, groups, fp_rows);
    if (n_int)
        hipLaunchKernelGGL(merged_ip_kernel<false>, dim3(N / KS_THREADS * groups, n_int), dim3(KS_THREADS), 0, stream,
                           rots, d_digits, digits_words(p, level), c0_base, c0_stride_r, dst_base, dst_stride, d_u,
                           p->d_mod, n, level, K, L, beta, p->alpha, p->logN, accumulate ? 1u : 0u, groups, int_rows);
    CKKS_LAUNCH_CHECK("merged_ip_kernel");
    return CKKS_OK;
}

template <bool RESC>
static void launch_moddown_tile(const ckks_params *p, const PtrPack &z, const PtrPack &out, const u64 *u, const u64 *w,
                                const u64 *bias, u32 n, u32 level, hipStream_t stream) {
    const u32 limbs = RESC ? level - 1 : level, tiles = p->N >> 12;
    const bool wide = wide_tiles((u64)tiles * limbs * n * 2);
    hipLaunchKernelGGL((wide ? moddown_tile_kernel<WIDE_RL, RESC> : moddown_tile_kernel<4, RESC>), dim3(tiles, limbs, n * 2),
                       dim3(tile_threads(wide)), 0, stream, z, out, u, w, bias, p->d_modf, p->d_mod, p->d_twf_fwd,
                       p->d_qlinv + (size_t)(level - 1) * p->L, level, p->K, p->logN);
}

// Merged giant step, part 2: out_r = z_r + ModDown(d_u[r]) for n <= ROT_BATCH ciphertexts [2][level][N]; d_u is consumed.
// d_w: n*2*level*N words of scratch.  out_r may be z_r, and is where moddown_mid_ok says no.
int moddown_add(ckks_params *p, u32 level, u64 *d_u, const u64 *const *z, u64 *const *out, u32 n, u64 *d_w,
                hipStream_t stream) {
    if (n == 0) return CKKS_OK;
    const u32 N = p->N, K = p->K, L = p->L, Wl = level + K;
    LimbIds ids;
    for (u32 t = 0; t < Wl; ++t) ids.id[t] = (uint8_t)(t < level ? SKIP_ROW : L + (t - level));
    const bool mid = moddown_mid_ok(p, level);      // the column passes of both transforms ride in the conversion
    int rc = launch_ntt(p, d_u, ids, Wl, n * 2 * Wl, true, stream, mid ? 1 : 3, true);
    if (rc) return rc;
    if (mid) {
        launch_moddown_mid(p, d_u, d_w, n, level, Wl, level, stream);
        CKKS_LAUNCH_CHECK("moddown_mid_kernel");
        p->limb_ntts += (u64)n * 2 * level;
        PtrPack zp, op;
        for (u32 r = 0; r < ROT_BATCH; ++r) {
            zp.p[r] = z[r < n ? r : 0];
            op.p[r] = out[r < n ? r : 0];
        }
        launch_moddown_tile<false>(p, zp, op, d_u, d_w, nullptr, n, level, stream);
        CKKS_LAUNCH_CHECK("moddown_tile_kernel");
        return CKKS_OK;
    }
    launch_moddown_conv(p, d_u, d_w, n, level, Wl, level, stream);
    CKKS_LAUNCH_CHECK("moddown_conv_kernel");
    for (u32 i = 0; i < level; ++i) ids.id[i] = (uint8_t)i;
    rc = launch_ntt(p, d_w, ids, level, n * 2 * level, false, stream);
    if (rc) return rc;
    ItemPack pack;
    for (u32 r = 0; r < ROT_BATCH; ++r) {
        SwitchItem &it = pack.it[r];
        it.digits = nullptr;
        it.c1 = nullptr;
        it.c0 = nullptr;                       // already folded in by switch_accumulate_merged
        it.key = nullptr;
        it.dst = out[r < n ? r : 0];
        it.add = z[r < n ? r : 0];
        it.galois_elt = 1;
        it.balanced = 0;
    }
    hipLaunchKernelGGL(moddown_final_kernel, dim3(N / KS_THREADS, level, n * 2), dim3(KS_THREADS), 0, stream, pack,
                       d_u, d_w, p->d_mod, level, K, p->logN);
    CKKS_LAUNCH_CHECK("moddown_final_kernel");
    return CKKS_OK;
}

// ModDown and rescale in one pass over the correction (merged giant step with CKKS_MATMUL_RESCALE):
//   out_r = rescale( z_r + ModDown(d_u[r]) + (bias_r, 0) ),   z_r [2][level][N] -> out_r [2][level-1][N],   n <= ROT_BATCH;
// bias [n][level][N] or null.  d_u is consumed; d_w: n*2*level*N words, d_t: n*2*N words of scratch.  Returns CKKS_E_INVAL if
// the fused kernels do not apply to this parameter set (the caller then brings down and rescales in two steps).
int moddown_rescale(ckks_params *p, u32 level, u64 *d_u, const u64 *const *z, const u64 *bias, u64 *const *out, u32 n,
                    u64 *d_w, u64 *d_t, hipStream_t stream) {
    if (n == 0) return CKKS_OK;
    if (!moddown_mid_ok(p, level) || level < 2) return CKKS_E_INVAL;
    const u32 N = p->N, K = p->K, L = p->L, Wl = level + K;
    PtrPack zp, op;
    for (u32 r = 0; r < ROT_BATCH; ++r) {
        zp.p[r] = z[r < n ? r : 0];
        op.p[r] = out[r < n ? r : 0];
    }
    LimbIds ids;
    for (u32 t = 0; t < Wl; ++t) ids.id[t] = (uint8_t)(t < level ? SKIP_ROW : L + (t - level));
    int rc = launch_ntt(p, d_u, ids, Wl, n * 2 * Wl, true, stream, 1, true);     // special limbs: inverse tile pass
    if (rc) return rc;
    hipLaunchKernelGGL(rescale_last_row_kernel, dim3(N / KS_THREADS, n * 2), dim3(KS_THREADS), 0, stream, zp, d_u, bias, d_t,
                       p->d_mod, level, K, N);
    CKKS_LAUNCH_CHECK("rescale_last_row_kernel");
    ids.id[0] = (uint8_t)(level - 1);
    rc = launch_ntt(p, d_t, ids, 1, n * 2, true, stream);
    if (rc) return rc;
    launch_moddown_mid(p, d_u, d_w, n, level, Wl, level, stream, d_t);
    CKKS_LAUNCH_CHECK("moddown_mid_kernel");
    p->limb_ntts += (u64)n * 2 * (level - 1);
    launch_moddown_tile<true>(p, zp, op, d_u, d_w, bias, n, level, stream);
    CKKS_LAUNCH_CHECK("moddown_tile_kernel");
    return CKKS_OK;
}

typedef decltype(&passb_final_kernel<true, true, 4, false>) passb_t;
template <bool CONV>
static passb_t passb_for(bool own_keys, bool wide, bool pair) {
    return own_keys ? (wide   ? passb_final_kernel<true, false, WIDE_RL, CONV>
                       : pair ? passb_final_kernel<true, true, 4, CONV>
                              : passb_final_kernel<true, false, 4, CONV>)
                    : (wide   ? passb_final_kernel<false, false, WIDE_RL, CONV>
                       : pair ? passb_final_kernel<false, true, 4, CONV>
                              : passb_final_kernel<false, false, 4, CONV>);
}

// n <= ROT_BATCH key switches from ready digits.  d_work: switch_scratch_words(level, n).
int switch_batch(ckks_params *p, u32 level, const SwitchItem *items, u32 n, u64 *d_work, hipStream_t stream) {
    if (n == 0) return CKKS_OK;
    if (n > ROT_BATCH) {
        set_error("switch_batch: %u items exceed one batch", n);
        return CKKS_E_INVAL;
    }
    const u32 N = p->N, K = p->K, L = p->L, Wl = level + K;
    const u32 beta = (level + p->alpha - 1) / p->alpha;
    ItemPack pack;
    const u32 n_groups = build_pack(items, n, pack);
    LimbIds ids;
    if (fast_ring(p) && beta <= MAX_BETA) {
        // inner product fused into the transforms on both sides of the base conversion
        u64 *y = d_work;                                   // [n][2][K][N]
        u64 *w = d_work + (size_t)n * 2 * K * N;           // [n][2][level][N]
        const u32 tiles = N >> 12;
        // at N = 2^12 the tile pass is the whole inverse transform and carries the (P/p_k)^-1 scaling itself
        const bool whole = p->logN == 12;
        const bool own_keys = n_groups == n;               // no two neighbouring items share a key
        // digits by 16-byte gathers above eight workgroups per CU: in tiles of 256 threads one rotation at level 1 of 2^16 (256
        // workgroups) took 85.8 us by 8-byte and 86.6 by 16-byte loads, two at level 1 94.9 and 95.7, four at level 24 (1024)
        // 299.7 and 300.2, 27 (6912) the same within the runs' 0.3 %; wide tiles, up to 512 workgroups, always 8-byte ones
        const bool ip_pair = tiles * n * 2 * K > 2048;
        const bool ip_wide = wide_tiles(tiles * n * 2 * K);
        const auto ip_intt = own_keys ? (ip_wide   ? ip_intt_kernel<true, false, WIDE_RL>
                                         : ip_pair ? ip_intt_kernel<true, true, 4>
                                                   : ip_intt_kernel<true, false, 4>)
                                      : (ip_wide   ? ip_intt_kernel<false, false, WIDE_RL>
                                         : ip_pair ? ip_intt_kernel<false, true, 4>
                                                   : ip_intt_kernel<false, false, 4>);
        hipLaunchKernelGGL(ip_intt, dim3(tiles, n * 2 * K), dim3(tile_threads(ip_wide)), 0, stream, pack, y, p->d_mod,
                           whole ? p->d_modf_dn : p->d_modf, p->d_tws_inv, p->d_twf_inv,
                           whole ? p->d_ninvs_dn : p->d_ninvs, n, level, K, L, beta, p->logN);
        CKKS_LAUNCH_CHECK("ip_intt_kernel");
        p->limb_ntts += (u64)n * 2 * K;
        int rc;
        // at N = 2^12 the base conversion rides in the last kernel: a row of the correction needs no other's columns
        const bool mid = moddown_mid_ok(p, level), conv = mid && whole;
        if (conv) {
            p->limb_ntts += (u64)n * 2 * level;
        } else if (mid) {
            // column passes of the inverse transform (special limbs) and of the forward one (correction) inside the
            // base conversion: one kernel, y read once, w written once
            launch_moddown_mid(p, y, w, n, level, K, 0u, stream);
            CKKS_LAUNCH_CHECK("moddown_mid_kernel");
            p->limb_ntts += (u64)n * 2 * level;
        } else {
            for (u32 k = 0; k < K; ++k) ids.id[k] = (uint8_t)(L + k);
            rc = launch_ntt(p, y, ids, K, n * 2 * K, true, stream, 2, true);
            if (rc) return rc;
            launch_moddown_conv(p, y, w, n, level, K, 0u, stream);
            CKKS_LAUNCH_CHECK("moddown_conv_kernel");
            for (u32 i = 0; i < level; ++i) ids.id[i] = (uint8_t)i;
            rc = launch_ntt(p, w, ids, level, n * 2 * level, false, stream, 1, false);
            if (rc) return rc;
        }
        // 16-byte gathers above three workgroups per CU: one rotation at 2^16, level 24 (768 workgroups) by 8-byte loads 165.0
        // us, by 16-byte ones 165.5; 24 switches at 2^14, level 5 (960) and the rest of their call 169 and 167; eight rotations
        // at 2^16, level 24 (6144) 496 and 493 (calls as long as they were then; wide tiles by 8-byte ones).
        const bool pair = tiles * n * 2 * level > 768;
        const bool wide = wide_tiles(tiles * n * 2 * level);
        const auto passb = conv ? passb_for<true>(own_keys, wide, pair) : passb_for<false>(own_keys, wide, pair);
        hipLaunchKernelGGL(passb, dim3(tiles, n * 2 * level), dim3(tile_threads(wide)), 0, stream, pack, conv ? y : w,
                           p->d_dn_mats, pad_pow2(K), p->d_mod, p->d_modf, p->d_tws_fwd, p->d_twf_fwd,
                           p->d_ninvs, n, level, K, L, beta, p->alpha, p->logN);
        CKKS_LAUNCH_CHECK("passb_final_kernel");
        return CKKS_OK;
    }
    u64 *u = d_work;
    u64 *w = d_work + (size_t)n * 2 * Wl * N;
    hipLaunchKernelGGL(inner_product_kernel, dim3(N / KS_THREADS, Wl, n_groups), dim3(KS_THREADS), 0, stream, pack, u,
                       p->d_mod, level, K, L, beta, p->alpha, p->logN);
    CKKS_LAUNCH_CHECK("inner_product_kernel");
    for (u32 t = 0; t < Wl; ++t) ids.id[t] = (uint8_t)(t < level ? SKIP_ROW : L + (t - level));
    int rc = launch_ntt(p, u, ids, Wl, n * 2 * Wl, true, stream, 3, true);
    if (rc) return rc;
    launch_moddown_conv(p, u, w, n, level, Wl, level, stream);
    CKKS_LAUNCH_CHECK("moddown_conv_kernel");
    for (u32 i = 0; i < level; ++i) ids.id[i] = (uint8_t)i;
    rc = launch_ntt(p, w, ids, level, n * 2 * level, false, stream);
    if (rc) return rc;
    hipLaunchKernelGGL(moddown_final_kernel, dim3(N / KS_THREADS, level, n * 2), dim3(KS_THREADS), 0, stream, pack,
                       u, w, p->d_mod, level, K, p->logN);
    CKKS_LAUNCH_CHECK("moddown_final_kernel");
    return CKKS_OK;
}

}  // namespace ckks

namespace ckks {

size_t rotate_hoisted_scratch_words(const ckks_params *P, u32 level, u32 n_steps) {
    const u32 batch = std::max<u32>(1, std::min<u32>(ROT_BATCH, n_steps));
    return digits_words(P, level) + (size_t)level * P->N + switch_scratch_words(P, level, batch);
}

int rotate_hoisted(ckks_params *P, const u64 *d_ct_in, u32 level, const int32_t *steps, u32 n_steps,
                   const ckks_gkey *const *keys, u64 *d_ct_out, size_t reserve_words, hipStream_t stream) {
    if (!P || !d_ct_in || (n_steps && (!steps || !d_ct_out))) {
        set_error("ckks_rotate_hoisted: null argument");
        return CKKS_E_INVAL;
    }
    if (level == 0 || level > P->L) {
        set_error("ckks_rotate_hoisted: level %u outside [1,%u]", level, P->L);
        return CKKS_E_LEVEL;
    }
    const u32 N = P->N;
    const size_t ctw = (size_t)2 * level * N;
    if (words_overlap(d_ct_in, ctw, d_ct_out, (size_t)n_steps * ctw)) {   // the switches gather from the input
        set_error("ckks_rotate_hoisted: d_ct_out overlaps d_ct_in");
        return CKKS_E_INVAL;
    }
    std::vector<SwitchItem> items;
    std::vector<u32> copies;
    for (u32 r = 0; r < n_steps; ++r) {
        u64 g;
        ckks_galois_elt(P, steps[r], &g);
        if (g == 1) {
            copies.push_back(r);
            continue;
        }
        if (P->K == 0) {
            set_error("ckks_rotate_hoisted: parameter set has no special primes");
            return CKKS_E_INVAL;
        }
        if (!keys || !keys[r]) {
            set_error("ckks_rotate_hoisted: step %d (index %u) has no key", steps[r], r);
            return CKKS_E_NOKEY;
        }
        if (keys[r]->params != P || keys[r]->galois_elt != g) {
            set_error("ckks_rotate_hoisted: key %u is for Galois element %llu, step %d needs %llu", r,
                      (unsigned long long)keys[r]->galois_elt, steps[r], (unsigned long long)g);
            return CKKS_E_INVAL;
        }
        SwitchItem it;
        it.digits = nullptr;
        it.c1 = d_ct_in + (size_t)level * N;
        it.c0 = d_ct_in;
        it.key = keys[r]->d_key;
        it.dst = d_ct_out + (size_t)r * ctw;
        it.galois_elt = g;
        it.add = nullptr;
        it.balanced = 0;
        items.push_back(it);
    }
    for (u32 r : copies)
        CKKS_HIP(hipMemcpyAsync(d_ct_out + (size_t)r * ctw, d_ct_in, ctw * sizeof(u64), hipMemcpyDeviceToDevice,
                                stream));
    if (items.empty()) return CKKS_OK;
    const u32 batch = std::min<u32>(ROT_BATCH, (u32)items.size());
    const size_t dig_w = digits_words(P, level), tmp_w = (size_t)level * N;
    int rc = P->ensure_scratch((reserve_words + dig_w + tmp_w + switch_scratch_words(P, level, batch)) * sizeof(u64),
                               stream);
    if (rc) return rc;
    u64 *d_digits = (u64 *)P->d_scratch + reserve_words, *d_tmp = d_digits + dig_w, *d_work = d_tmp + tmp_w;
    const u64 *c1 = d_ct_in + (size_t)level * N;
    rc = decompose(P, &c1, 1, level, d_digits, d_tmp, stream);
    if (rc) return rc;
    for (auto &it : items) it.digits = d_digits;
    for (size_t done = 0; done < items.size(); done += batch) {
        u32 n = (u32)std::min<size_t>(batch, items.size() - done);
        rc = switch_batch(P, level, items.data() + done, n, d_work, stream);
        if (rc) return rc;
    }
    return CKKS_OK;
}

}  // namespace ckks

using namespace ckks;

extern "C" {

int ckks_galois_key_load(const ckks_params_t *P, uint64_t galois_elt, const uint64_t *d_key, void *stream,
                         ckks_gkey_t **out) {
    if (!out) {
        set_error("ckks_galois_key_load: out is null");
        return CKKS_E_INVAL;
    }
    *out = nullptr;
    if (!P || !d_key) {
        set_error("ckks_galois_key_load: null argument");
        return CKKS_E_INVAL;
    }
    if (P->K == 0) {
        set_error("ckks_galois_key_load: parameter set has no special primes");
        return CKKS_E_INVAL;
    }
    if (!(galois_elt & 1) || galois_elt >= 2ull * P->N || galois_elt == 1) {
        set_error("ckks_galois_key_load: %llu is not a non-trivial Galois element", (unsigned long long)galois_elt);
        return CKKS_E_INVAL;
    }
    ckks_gkey *k = new ckks_gkey();
    k->params = P;
    k->galois_elt = galois_elt;
    size_t rows = (size_t)P->dnum * 2 * P->W;
    hipError_t e = hipMalloc((void **)&k->d_key, rows * P->N * sizeof(u64));
    if (e != hipSuccess) {
        delete k;
        return hip_fail(e, "hipMalloc(key)");
    }
    hipLaunchKernelGGL(key_form_kernel, dim3(P->N / (4 * KS_THREADS), (u32)rows), dim3(KS_THREADS), 0, (hipStream_t)stream,
                       d_key, k->d_key, P->d_mod, P->d_pinv, P->L, P->W, P->N);
    e = hipGetLastError();
    if (e != hipSuccess) {
        hipFree(k->d_key);
        delete k;
        return hip_fail(e, "key_form_kernel");
    }
    *out = k;
    return CKKS_OK;
}

int ckks_galois_key_adopt(const ckks_params_t *P, uint64_t galois_elt, uint64_t *d_key, void *stream,
                          ckks_gkey_t **out) {
    if (!out) {
        set_error("ckks_galois_key_adopt: out is null");
        return CKKS_E_INVAL;
    }
    *out = nullptr;
    if (!P || !d_key || P->K == 0) {
        set_error("ckks_galois_key_adopt: null argument or no special primes");
        return CKKS_E_INVAL;
    }
    if (!(galois_elt & 1) || galois_elt >= 2ull * P->N || galois_elt == 1) {
        set_error("ckks_galois_key_adopt: %llu is not a non-trivial Galois element", (unsigned long long)galois_elt);
        return CKKS_E_INVAL;
    }
    const size_t rows = (size_t)P->dnum * 2 * P->W;
    // each thread reads the residues it writes before it writes them: in place is safe
    hipLaunchKernelGGL(key_form_kernel, dim3(P->N / (4 * KS_THREADS), (u32)rows), dim3(KS_THREADS), 0, (hipStream_t)stream,
                       d_key, d_key, P->d_mod, P->d_pinv, P->L, P->W, P->N);
    CKKS_LAUNCH_CHECK("key_form_kernel");
    ckks_gkey *k = new ckks_gkey();
    k->params = P;
    k->galois_elt = galois_elt;
    k->d_key = d_key;
    k->owned = false;
    *out = k;
    return CKKS_OK;
}

int ckks_relin_key_load(const ckks_params_t *P, const uint64_t *d_key, void *stream, ckks_gkey_t **out) {
    if (!out) {
        set_error("ckks_relin_key_load: out is null");
        return CKKS_E_INVAL;
    }
    *out = nullptr;
    if (!P || !d_key || P->K == 0) {
        set_error("ckks_relin_key_load: null argument or no special primes");
        return CKKS_E_INVAL;
    }
    ckks_gkey *k = new ckks_gkey();
    k->params = P;
    k->galois_elt = 1;   // no automorphism: the key switches from s^2
    size_t rows = (size_t)P->dnum * 2 * P->W;
    hipError_t e = hipMalloc((void **)&k->d_key, rows * P->N * sizeof(u64));
    if (e != hipSuccess) {
        delete k;
        return hip_fail(e, "hipMalloc(key)");
    }
    hipLaunchKernelGGL(key_form_kernel, dim3(P->N / (4 * KS_THREADS), (u32)rows), dim3(KS_THREADS), 0, (hipStream_t)stream,
                       d_key, k->d_key, P->d_mod, P->d_pinv, P->L, P->W, P->N);
    e = hipGetLastError();
    if (e != hipSuccess) {
        hipFree(k->d_key);
        delete k;
        return hip_fail(e, "key_form_kernel");
    }
    *out = k;
    return CKKS_OK;
}

int ckks_ctmul(ckks_params_t *P, const uint64_t *d_ct_a, const uint64_t *d_ct_b, uint32_t level,
               const ckks_gkey_t *relin_key, uint64_t *d_ct_out, void *stream_) {
    hipStream_t stream = (hipStream_t)stream_;
    if (!P || !d_ct_a || !d_ct_b || !d_ct_out) {
        set_error("ckks_ctmul: null argument");
        return CKKS_E_INVAL;
    }
    if (level == 0 || level > P->L) {
        set_error("ckks_ctmul: level %u outside [1,%u]", level, P->L);
        return CKKS_E_LEVEL;
    }
    if (!relin_key) {
        set_error("ckks_ctmul: no relinearisation key");
        return CKKS_E_NOKEY;
    }
    if (relin_key->params != P || relin_key->galois_elt != 1) {
        set_error("ckks_ctmul: the key is not a relinearisation key of this parameter set");
        return CKKS_E_INVAL;
    }
    const u32 N = P->N;
    if (words_overlap(d_ct_out, (size_t)2 * level * N, d_ct_a, (size_t)2 * level * N) ||
        words_overlap(d_ct_out, (size_t)2 * level * N, d_ct_b, (size_t)2 * level * N)) {
        set_error("ckks_ctmul: d_ct_out overlaps an input");
        return CKKS_E_INVAL;
    }
    const size_t dig_w = digits_words(P, level), lim_w = (size_t)level * N;
    int rc = P->ensure_scratch((dig_w + 2 * lim_w + switch_scratch_words(P, level, 1)) * sizeof(u64), stream);
    if (rc) return rc;
    u64 *d_digits = (u64 *)P->d_scratch, *d_tmp = d_digits + dig_w, *d_t2 = d_tmp + lim_w, *d_work = d_t2 + lim_w;
    bool one = fast_ring(P);                                 // see tensor_intt_kernel
    for (u32 i = 0; i < level && P->logN < 15; ++i) one = one && (P->mod[i] >> 50) == 0;
    if (one) {
        const LevelTables *lt = nullptr;
        rc = P->level_tables(level, &lt);
        if (rc) return rc;
        const bool wide = wide_tiles((u64)(N >> 12) * level);
        hipLaunchKernelGGL(wide ? tensor_intt_kernel<WIDE_RL> : tensor_intt_kernel<4>, dim3(N >> 12, level),
                           dim3(tile_threads(wide)), 0, stream, d_ct_a, d_ct_b, d_ct_out, d_t2, d_tmp, P->d_mod,
                           decompose_modf(P, lt), P->d_tws_inv, P->d_twf_inv, P->d_ninvs, level, P->logN);
        CKKS_LAUNCH_CHECK("tensor_intt_kernel");
        P->limb_ntts += level;
        rc = decompose_from_tmp(P, lt, 1, d_digits, d_tmp, stream, false);
    } else {
        hipLaunchKernelGGL(tensor_kernel, dim3(N / KS_THREADS, level), dim3(KS_THREADS), 0, stream, d_ct_a, d_ct_b,
                           d_ct_out, d_t2, P->d_mod, level, N);
        CKKS_LAUNCH_CHECK("tensor_kernel");
        const u64 *c1 = d_t2;
        rc = decompose(P, &c1, 1, level, d_digits, d_tmp, stream);
    }
    if (rc) return rc;
    SwitchItem it;
    it.digits = d_digits;
    it.c1 = d_t2;
    it.c0 = nullptr;            // (t0, t1) are already in the output: the switch only adds ModDown(...)
    it.key = relin_key->d_key;
    it.dst = d_ct_out;
    it.galois_elt = 1;
    it.add = d_ct_out;
    it.balanced = 0;
    return switch_batch(P, level, &it, 1, d_work, stream);
}

void ckks_galois_key_destroy(ckks_gkey_t *key) {
    if (!key) return;
    if (key->owned) hipFree(key->d_key);
    delete key;
}

int ckks_rotate_hoisted(ckks_params_t *P, const uint64_t *d_ct_in, uint32_t level, const int32_t *steps,
                        uint32_t n_steps, const ckks_gkey_t *const *keys, uint64_t *d_ct_out, void *stream_) {
    return rotate_hoisted(P, d_ct_in, level, steps, n_steps, keys, d_ct_out, 0, (hipStream_t)stream_);
}

}  // extern "C"
