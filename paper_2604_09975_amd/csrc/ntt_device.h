// Device-side building blocks of the radix-16 NTT (N = 2^12 .. 2^17), shared by the transform kernels
// and by the key-switch kernels that fuse other work into a transform pass.
#pragma once
#include "ckks_internal.h"

namespace ckks {

constexpr u32 NTT_THREADS = 256;

// A tile of 4096 residues and the workgroup that transforms it, 2^RL residues a thread: 256 threads with 16 residues each
// (RL = 4), or 1024 with 4 (RL = WIDE_RL) in launches of few workgroups.
// LDS slot of tile element i: one padding word after every 2^RL elements.  The access patterns of the tile pass
// (residues 2^(12-RL) apart down to 2^RL consecutive ones per thread) then fall on distinct banks but for a few pairs, and,
// unlike an XOR fold, every slot a thread touches is its base slot plus a compile-time offset: no address registers, which
// is what brings the pass from 130 to under 100 vector registers.  A tile takes 34 KiB (RL = 2: 40); four fit a CU.
template <u32 RL>
struct Tile {
    static constexpr u32 R = 1u << RL, THREADS = 4096u >> RL, WORDS = 4096 + (4096u >> RL), ROUNDS = 12 / RL;
    // WAVE: in the rounds whose residues lie at most 64 apart (all but the first at RL = 3, all but the first two at RL = 2), and
    // so at the pass's LDS end, a wavefront touches 64 R consecutive elements of its own only.  The exchanges among rounds
    // with more between their residues are the workgroup's (Round::BEHIND, Round::FRONT).
    static constexpr bool WAVE = RL < 4;
    static_assert(12 % RL == 0 && (!WAVE || (4096u >> (RL * ROUNDS) << RL) <= 64 * R), "the last round is a wavefront's own");
    static __device__ __forceinline__ u32 slot(u32 i) { return i + (i >> RL); }
    // the i-th single element and the i-th pair of elements of a thread at the pass's LDS end
    static __device__ __forceinline__ u32 one(u32 tid, u32 i) {
        return WAVE ? (tid & ~63u) * R + (tid & 63u) + 64 * i : tid + THREADS * i;
    }
    static __device__ __forceinline__ u32 pair(u32 tid, u32 i) {
        return WAVE ? (tid & ~63u) * R + (tid & 63u) * 2 + 128 * i : 2 * (tid + THREADS * i);
    }
};

// A launch of few workgroups lasts as long as one of them, and with 256 threads that is one wavefront per SIMD waiting for
// its operands, then for each round's twiddles and exchange.  With 1024 threads four wavefronts share the wait, every load
// of the operands is on its way at once, and the operands of a key switch's last pass arrive during its transform.
// 512 workgroups of 1024 threads are two per CU, which is what runs at a time of the kernels of up to 64 registers (the
// transforms, gather_intt, the rescales).  us with 256 threads, with wide tiles up to 512 and up to 1024 workgroups (calls as
// long as they were when the line was drawn):
// ip_intt_kernel of 7 switches at 2^12 (14 workgroups) 19.3 -> 11.5; whole calls: toy projection at 2^12 145 / 112 / 112,
// product and rescale at 2^15 (12 + 4 primes) 130 / 104 / 104, one rotation at 2^16, level 17 (544 and 928 workgroups in two of
// its kernels) 154 / 137 / 143, 24 switches and 12 rescales at 2^14 (960 in one) 165 / 146 / 155.  512 threads with 8
// residues: 113, 105, 140, 151.
// ip_intt_kernel (76 registers) and passb_final_kernel (103 to 106) run one such workgroup per CU, so from 257 on there are two
// rounds of them.  The first is the faster one all the same: calls of 320 / 480 / 512 workgroups in it (five switches at 2^15,
// 30 at 2^14, two at 2^16) 83.7 / 127.0 / 87.3 us, by 256 threads from 257 on 87.6 / 133.4 / 90.1.  The second is not always,
// 0.5 to 2.9 % of a call either way: one rotation at 2^16, levels 9 / 12 / 16 (288 / 384 / 512 in it) 91.6 / 93.2 / 96.6, by 256
// threads 90.0 / 92.4 / 95.5, three at 2^15, level 6 (288) 70.1 and 68.0; two at 2^16, level 8 (512) 87.3 and 87.9, fifteen at
// 2^14, level 4 (480) 69.6 and 71.7.
constexpr u32 WIDE_RL = 2;
inline bool wide_tiles(u64 workgroups) { return workgroups <= 512; }
inline u32 tile_threads(bool wide) { return wide ? 1024 : 256; }

// After the exchange through LDS of data that goes no further than SPAN threads.  Within a wavefront LDS instructions
// execute in order, and only the compiler has to be kept from moving them.
template <u32 SPAN>
__device__ __forceinline__ void exchange_sync() {
    if constexpr (SPAN > 64) {
        __syncthreads();
    } else {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
}

// Integer butterflies for primes that neither fit the fp64 scheme nor fold (FieldPm): lazy values and
// twiddles with a precomputed quotient.  A twiddle is the pair (w, w') with w' = floor(w * 2^64 / q); for any 64-bit
// y, y*w - floor(y*w' / 2^64) * q lies in [0, 2q) and is congruent to y*w: one high product and two low products,
// no correction step.  Forward values live in [0, 4q), inverse values in [0, 2q) (q < 2^62 keeps 4q in a word);
// out() brings a value back to [0, q).
struct TwInt {
    u64 w, ws;
};

struct FieldInt {
    typedef u64 T;
    template <bool U> using W = TwInt;
    static constexpr bool BOUNDED = false;
    u64 q, q2;
    const ulonglong2 *tw;
    TwInt n0, n1;
    __device__ __forceinline__ T in(u64 x) const { return x; }
    __device__ __forceinline__ u64 out(T x) const {
        if (x >= q2) x -= q2;
        if (x >= q) x -= q;
        return x;
    }
    __device__ __forceinline__ u64 bits(T x) const { return x; }
    __device__ __forceinline__ u64 half(T x) const { return x; }
    __device__ __forceinline__ T from_bits(u64 x) const { return x; }
    template <bool U>
    __device__ __forceinline__ TwInt twid(u32 idx, u32 k) const {
        const ulonglong2 t = (tw + idx)[k];
        return TwInt{t.x, t.y};
    }
    __device__ __forceinline__ void norm(T &) const {}
    __device__ __forceinline__ T mul(T y, const TwInt &w) const { return y * w.w - mul_hi(y, w.ws) * q; }   // [0, 2q)
    __device__ __forceinline__ void fwd(T &x, T &y, const TwInt &w) const {
        if (x >= q2) x -= q2;
        const T v = mul(y, w);
        y = x - v + q2;
        x = x + v;
    }
    __device__ __forceinline__ void inv(T &x, T &y, const TwInt &w) const {
        T s = x + y;
        if (s >= q2) s -= q2;
        y = mul(x - y + q2, w);
        x = s;
    }
    __device__ __forceinline__ void inv_last(T &x, T &y) const {
        const T s = x + y, d = x - y + q2;
        x = mul(s, n0);
        y = mul(d, n1);
    }
};

// Integer butterflies for primes q = 2^b - c, 51 <= b <= 60, 0 < c < 2^(b-35): signed lazy values below 8 q in magnitude, and
// a reduction that folds at 2^b = c (mod q) instead of multiplying by a quotient.  A value y = yh 2^32 + yl (halves signed) is
// multiplied by w as yl w + yh (2^32 w mod q); both factors are stored balanced and cut at 2^s, s = b - 32, into signed halves,
//   p1 = yl w1 + yh v1 + 2^31,   p0 = yl w0 + yh v0 - 2^(b-1),   y w = p1 2^s + p0   (mod q),
// |p1| < 2^63 as |yl|, |w1|, |v1| <= 2^31 and |yh| < 2^31 - 1, |p0| <= 2^b; and with p1 = h 2^32 + l, p1 2^s = h 2^b + l 2^s:
//   y w = h c + (p0 + l 2^s).
// Six 32 x 32-bit multiply-adds and an addition (the rounding of y's halves).  |y w| <= (25/32 + 9/256 |y|/q) q: 2^(b-2) (1 +
// |yh| / 2^31) from p0, 2^(b-1) from l, c 2^30 (1 + |yh| / 2^31) from h.
// A butterfly is 13 issue slots where one with a quotient per product (FieldInt) is 30 and an fp64 one 10 (measured, slots of
// one 32-bit operation at 2.4 GHz; 16 wavefronts per CU).
// Launches before and after: ip_intt_kernel of 27 switches at 2^16 340 -> 284 us, of 24 switches that share keys 244 -> 208,
// one 16.2 -> 14.1; merged_tile_kernel of the QKV projection 1.82 -> 1.58 ms; three rows of four limbs at 2^13, inverse, 13.3
// -> 11.4 us.
// The multiply-adds are written out: the compiler takes products of halves of a 64-bit word apart into unsigned ones and
// corrections (25 slots per butterfly).  U: the twiddle is the same for the wavefront, and comes in scalar registers.
template <bool U>
struct TwPm {
    int w0, w1, v0, v1;
};

struct FieldPm {
    typedef int64_t T;
    template <bool U> using W = TwPm<U>;
    // bounds in units of q / 256 (a canonical value: 256): of a product of a value bounded by b, of normalised values and of
    // those that the rounds of an inverse pass leave; and of every value, sum and difference: below 7.5 2^b, where norm ends for
    // b = 60 (mul takes up to 2^63 - 2^33)
    static constexpr bool BOUNDED = true;
    static constexpr u32 NORMED = 129, INV_BASE = 264, LIMIT = 1919;
    static constexpr u32 product(u32 b) { return 201 + (9 * b + 255) / 256; }
    u64 q, q8;
    int64_t r31, mid;                       // 2^31 and -2^(b-1)
    int c;
    u32 s, p2s;                             // s and 2^s
    const int4 *tw;
    TwPm<true> n0, n1;
    __device__ __forceinline__ T in(u64 x) const { return (T)x; }
    __device__ __forceinline__ u64 out(T x) const {
        const u64 y = (u64)x + q8;          // [0, 16 q)
        const u32 hi = (u32)(y >> 32);
        const u64 r = (u64)(hi >> s) * (u32)c + ((u64)(hi & (p2s - 1)) << 32 | (u32)y);   // below 2 q
        return r >= q ? r - q : r;
    }
    __device__ __forceinline__ u64 bits(T x) const { return (u64)x; }
    __device__ __forceinline__ u64 half(T x) const {
        norm(x);
        return (u64)x;
    }
    __device__ __forceinline__ T from_bits(u64 x) const { return (T)x; }
    template <bool U>
    __device__ __forceinline__ TwPm<U> twid(u32 idx, u32 k) const {
        const int4 t = (tw + idx)[k];
        return TwPm<U>{t.x, t.y, t.z, t.w};
    }
    // x -> x - round(x / 2^b) q, at most 2^(b-1) + |x / 2^b| c + c / 2 (from fold30: 2^(b-1) + 2^26).  hi - lo fits 32 bits below 7.5 2^60
    __device__ __forceinline__ void norm(T &x) const {
        const int hi = (int)(x >> 32), lo = __builtin_amdgcn_sbfe(hi, 0, s);
        const int64_t y = (int64_t)((u64)(u32)lo << 32 | (u32)x);
        u64 co;
        asm("v_mad_i64_i32 %0, %1, %2, %3, %4" : "=v"(x), "=s"(co) : "v"((hi - lo) >> s), "s"(c), "v"(y));
    }
    template <bool U>
    __device__ __forceinline__ T mul(T y, const TwPm<U> &w) const {
        const int yl = (int)y, yh = (int)((y + r31) >> 32);
        int64_t p0, p1;
        u64 co;
#define PM_PARTS                                                                              \
    "v_mad_i64_i32 %1, %2, %3, %6, %9\n\tv_mad_i64_i32 %0, %2, %3, %5, %10\n\t"               \
    "v_mad_i64_i32 %1, %2, %4, %8, %1\n\tv_mad_i64_i32 %0, %2, %4, %7, %0"
        if constexpr (U)
            asm(PM_PARTS : "=&v"(p0), "=&v"(p1), "=&s"(co)
                : "v"(yl), "v"(yh), "s"(w.w0), "s"(w.w1), "s"(w.v0), "s"(w.v1), "v"(r31), "v"(mid));
        else
            asm(PM_PARTS : "=&v"(p0), "=&v"(p1), "=&s"(co)
                : "v"(yl), "v"(yh), "v"(w.w0), "v"(w.w1), "v"(w.v0), "v"(w.v1), "v"(r31), "v"(mid));
#undef PM_PARTS
        T r;
        asm("v_mad_u64_u32 %0, %1, %3, %5, %6\n\tv_mad_i64_i32 %0, %1, %2, %4, %0"
            : "=&v"(r), "=&s"(co)
            : "v"((int)(p1 >> 32)), "v"((u32)p1), "s"(c), "s"(p2s), "v"(p0));
        return r;
    }
    // lo + hi 2^30 for lo < 2^59, hi < 2^(b-1): normalised, or canonical
    __device__ __forceinline__ u64 fold30(u64 lo, u64 hi, bool canonical) const {
        const u32 sh = s + 2, top = (u32)(hi >> sh), low = (u32)hi & ((1u << sh) - 1);      // hi 2^30 = top 2^b + low 2^30
        T x = (T)((u64)top * (u32)c + lo + ((u64)low << 30));                               // below 2^61
        norm(x);
        return canonical ? out(x) : (u64)x;
    }
    template <bool U>
    __device__ __forceinline__ void fwd(T &x, T &y, const TwPm<U> &w) const {
        const T v = mul(y, w);
        y = x - v;
        x = x + v;
    }
    template <bool U>
    __device__ __forceinline__ void inv(T &x, T &y, const TwPm<U> &w) const {
        const T s = x + y;
        y = mul(x - y, w);
        x = s;
    }
    __device__ __forceinline__ void inv_last(T &x, T &y) const {
        const T s = x + y, d = x - y;
        x = mul(s, n0);
        y = mul(d, n1);
    }
};

// Exact integer arithmetic in doubles for q < 2^50.  mul(a, w) returns r = a*w - c*q with
// c = rint(a*w/q) computed in floating point: |r| <= (1/2 + 3|a|/2^53) q, exact as long as
// |a| <= 2^52.  Sums stay exact below 2^53.  norm() brings a value back to |x| <= q/2.
struct FieldFp {
    typedef double T;
    template <bool U> using W = double;
    static constexpr bool BOUNDED = false;
    double q, u, n0, n1;
    const double *tw;
    __device__ __forceinline__ T in(u64 x) const {
        return __longlong_as_double((long long)(x | 0x4330000000000000ull)) - 4503599627370496.0;
    }
    __device__ __forceinline__ void norm(T &x) const {
        const double c = rint(x * u);
        x = fma(-c, q, x);
    }
    __device__ __forceinline__ u64 out(T x) const {
        norm(x);
        if (x < 0) x += q;
        return (u64)__double_as_longlong(x + 4503599627370496.0) & 0x000fffffffffffffull;
    }
    __device__ __forceinline__ u64 bits(T x) const { return (u64)__double_as_longlong(x); }
    __device__ __forceinline__ u64 half(T x) const { return (u64)__double_as_longlong(x); }
    __device__ __forceinline__ T from_bits(u64 x) const { return __longlong_as_double((long long)x); }
    template <bool U>
    __device__ __forceinline__ double twid(u32 idx, u32 k) const { return (tw + idx)[k]; }   // entry idx + k; k constant: wide loads
    __device__ __forceinline__ T mul(T a, T w) const {
        const double h = a * w;
        const double l = fma(a, w, -h);
        const double c = rint(h * u);
        const double d = fma(-c, q, h);
        return d + l;
    }
    __device__ __forceinline__ void fwd(T &x, T &y, T w) const {
        const T v = mul(y, w);
        y = x - v;
        x = x + v;
    }
    __device__ __forceinline__ void inv(T &x, T &y, T w) const {
        const T s = x + y;
        y = mul(x - y, w);
        x = s;
    }
    __device__ __forceinline__ void inv_last(T &x, T &y) const {
        const T s = x + y, d = x - y;
        x = mul(s, n0);
        y = mul(d, n1);
    }
};

// LOGR stages on the 2^LOGR values a thread holds.  The group is node `nb` of stage s0; at stage
// s0 + t it covers nodes (nb << t) + k, k < 2^t, and values j, j + (2^LOGR >> t + 1) pair up.
// fp64 bounds: a product is below 0.9 q (a factor below 4q) or 0.7 q (below q), so four forward stages take a
// normalised value (q/2) to 4 q = 2^52; an inverse stage doubles a value and hands the difference, twice as large, to
// the product: two of them between normalisations.
// A bounded field (FieldPm) is normalised where the next sum could pass its limit; the bounds are known at compile time.
// IN: bound of the values of a forward group (radix_out gives the next one's); canonical ones by default.
template <class F>
constexpr u32 radix_out(u32 in, u32 stages) {
    if constexpr (F::BOUNDED)
        for (u32 t = 0; t < stages; ++t) {
            if (in + F::product(in) > F::LIMIT) in = F::NORMED;
            in += F::product(in);
        }
    return in;
}
constexpr u32 CANONICAL = 256;
// S0: stages since values were normalised
template <u32 LOGR, u32 IN, u32 S0 = 0, class F, class Tw>
__device__ __forceinline__ void radix_fwd_by(const F &f, typename F::T (&v)[1u << LOGR], Tw tw) {
    constexpr u32 R = 1u << LOGR;
    u32 bound = IN;
#pragma unroll
    for (u32 t = 0; t < LOGR; ++t) {
        bool norm = (S0 + t) % 4 == 0;
        if constexpr (F::BOUNDED) {
            norm = bound + F::product(bound) > F::LIMIT;
            if (norm) bound = F::NORMED;
            bound += F::product(bound);
        }
        if (norm) {
#pragma unroll
            for (u32 j = 0; j < R; ++j) f.norm(v[j]);
        }
        const u32 g = R >> (t + 1);
#pragma unroll
        for (u32 k = 0; k < (1u << t); ++k) {
            const auto w = tw(t, k);
#pragma unroll
            for (u32 i = 0; i < g; ++i) f.fwd(v[k * 2 * g + i], v[k * 2 * g + i + g], w);
        }
    }
}
template <u32 LOGR, bool U = true, u32 IN = CANONICAL, class F>
__device__ __forceinline__ void radix_fwd(const F &f, typename F::T (&v)[1u << LOGR], u32 s0, u32 nb) {
    radix_fwd_by<LOGR, IN>(f, v, [&](u32 t, u32 k) { return f.template twid<U>((1u << (s0 + t)) + (nb << t), k); });
}

// last: the group's first stage (t = 0) ends the transform and folds in N^-1.  MORE: another group follows before the values
// leave the field
template <u32 LOGR, bool MORE, class F, class Tw>
__device__ __forceinline__ void radix_inv_by(const F &f, typename F::T (&v)[1u << LOGR], Tw tw, bool last) {
    constexpr u32 R = 1u << LOGR;
    u32 bound[R];
    if constexpr (F::BOUNDED) {
#pragma unroll
        for (u32 j = 0; j < R; ++j) bound[j] = F::INV_BASE;
    }
#pragma unroll
    for (int t = (int)LOGR - 1; t >= 0; --t) {
        const u32 g = R >> (t + 1);
        if constexpr (F::BOUNDED) {
#pragma unroll
            for (u32 k = 0; k < (1u << t); ++k)
#pragma unroll
                for (u32 i = 0; i < g; ++i) {
                    const u32 x = k * 2 * g + i, y = x + g;
                    if (bound[x] + bound[y] > F::LIMIT) {
                        f.norm(v[x]);
                        f.norm(v[y]);
                        bound[x] = bound[y] = F::NORMED;
                    }
                    bound[x] += bound[y];
                    bound[y] = F::product(bound[x]);
                }
        } else if (((int)LOGR - 1 - t) % 2 == 0) {
#pragma unroll
            for (u32 j = 0; j < R; ++j) f.norm(v[j]);
        }
        if (t == 0 && last) {
#pragma unroll
            for (u32 i = 0; i < R / 2; ++i) f.inv_last(v[i], v[i + R / 2]);
        } else {
#pragma unroll
            for (u32 k = 0; k < (1u << t); ++k) {
                const auto w = tw((u32)t, k);
#pragma unroll
                for (u32 i = 0; i < g; ++i) f.inv(v[k * 2 * g + i], v[k * 2 * g + i + g], w);
            }
        }
    }
    if constexpr (F::BOUNDED && MORE) {
#pragma unroll
        for (u32 j = 0; j < R; ++j)
            if (bound[j] > F::INV_BASE) f.norm(v[j]);
    }
}
template <u32 LOGR, bool U, bool MORE, class F>
__device__ __forceinline__ void radix_inv(const F &f, typename F::T (&v)[1u << LOGR], u32 s0, u32 nb, bool last) {
    radix_inv_by<LOGR, MORE>(f, v, [&](u32 t, u32 k) { return f.template twid<U>((1u << (s0 + t)) + (nb << t), k); }, last);
}

// Between the two passes of a transform (N above 2^12) a row holds the field's own values as the first pass leaves them,
// half(): doubles of up to 4 q, lazy integers, normalised ones on primes that fold.  The second pass starts by normalising
// doubles anyway; canonical residues there cost a conversion each way, ten instructions of the hundred of a tile pass.
//
// pass B: the last 12 stages act inside aligned runs of 4096 consecutive residues, one workgroup per run, in 12 / RL
// rounds of RL stages with an LDS exchange between them.  In round r a thread holds 2^RL residues S = 4096 >> RL (r + 1)
// apart, those of block tid / S from tid % S on:
//   RL = 4: 256 apart (2 KiB runs in global memory), 16 apart, consecutive;  RL = 2: 1024, 256, 64, 16, 4 apart, consecutive.
// The exchange behind round r stays among the S threads of a block: within a wavefront from S = 64 down.
// For N = 2^12 this is the whole transform.  The passes come in halves so that callers can put their own code
// between global memory and LDS.  LDS slot of residue e of the tile: lds[Tile<RL>::slot(e)].
// RL = WIDE_RL: each round's twiddles are loaded a round ahead, as there are few wavefronts to hide the wait; larger RL have
// none of the registers that takes.
template <u32 RL, u32 RD>
struct Round {
    static constexpr u32 S = 4096u >> (RL * (RD + 1));
    static constexpr bool UNIFORM = S >= 64;                         // a wavefront's residues are of one node
    static constexpr u32 BEHIND = RL < 4 ? S : (4096u >> RL);        // threads that the exchange behind the round spans
    static constexpr u32 FRONT = RL < 4 ? S << RL : (4096u >> RL);   // and the one in front of it
    static __device__ __forceinline__ u32 first() { return threadIdx.x / S * (S << RL) + threadIdx.x % S; }
    static __device__ __forceinline__ u32 elem(u32 j) { return first() + j * S; }
    // Tile<RL>::slot(elem(j)), written so that the j are constant offsets: S is 1 or a multiple of 2^RL
    static __device__ __forceinline__ u32 slot(u32 j) { return Tile<RL>::slot(first()) + j * (S + (S >> RL)); }
    static __device__ __forceinline__ u32 node(u32 tile) {
        const u32 blk = S >= 64 ? __builtin_amdgcn_readfirstlane(threadIdx.x / S) : threadIdx.x / S;
        return (tile << (RL * RD)) + blk;
    }
    static __device__ __forceinline__ u32 stage(u32 logN) { return logN - 12 + RL * RD; }
};

template <u32 RL, u32 RD, class F>
struct Twids {
    typename F::template W<(RD < 12 / RL) && Round<RL, RD>::UNIFORM> w[RL == WIDE_RL ? (1u << RL) - 1 : 1];
};
template <u32 RL, u32 RD, class F>
__device__ __forceinline__ void load_twids(const F &f, u32 logN, u32 tile, Twids<RL, RD, F> &tw) {
    if constexpr (RL == WIDE_RL && RD < 12 / RL) {
        const u32 s0 = Round<RL, RD>::stage(logN), nb = Round<RL, RD>::node(tile);
#pragma unroll
        for (u32 t = 0; t < RL; ++t)
#pragma unroll
            for (u32 k = 0; k < (1u << t); ++k)
                tw.w[(1u << t) - 1 + k] = f.template twid<Round<RL, RD>::UNIFORM>((1u << (s0 + t)) + (nb << t), k);
    }
}
template <u32 RL, u32 RD, class F>
__device__ __forceinline__ void round_fwd(const F &f, typename F::T (&v)[1u << RL], u32 logN, u32 tile,
                                          const Twids<RL, RD, F> &tw) {
    constexpr u32 IN = radix_out<F>(CANONICAL, RL * RD);
    if constexpr (RL == WIDE_RL)
        radix_fwd_by<RL, IN, RL * RD>(f, v, [&](u32 t, u32 k) { return tw.w[(1u << t) - 1 + k]; });
    else
        radix_fwd<RL, Round<RL, RD>::UNIFORM, IN>(f, v, Round<RL, RD>::stage(logN), Round<RL, RD>::node(tile));
}
template <u32 RL, u32 RD, class F>
__device__ __forceinline__ void round_inv(const F &f, typename F::T (&v)[1u << RL], u32 logN, u32 tile,
                                          const Twids<RL, RD, F> &tw, bool last) {
    if constexpr (RL == WIDE_RL)
        radix_inv_by<RL, (RD > 0)>(f, v, [&](u32 t, u32 k) { return tw.w[(1u << t) - 1 + k]; }, last);
    else
        radix_inv<RL, Round<RL, RD>::UNIFORM, (RD > 0)>(f, v, Round<RL, RD>::stage(logN), Round<RL, RD>::node(tile), last);
}

// forward rounds from RD on, LDS to LDS
template <bool RAW, u32 RL, u32 RD, class F>
__device__ __forceinline__ void fwd_rounds(const F &f, u32 logN, u32 tile, u64 *lds, const Twids<RL, RD, F> &tw) {
    typedef Tile<RL> TL;
    typedef Round<RL, RD> RN;
    Twids<RL, RD + 1, F> next;
    load_twids<RL, RD + 1>(f, logN, tile, next);
    typename F::T v[TL::R];
#pragma unroll
    for (u32 j = 0; j < TL::R; ++j) v[j] = f.from_bits(lds[RN::slot(j)]);
    round_fwd<RL, RD>(f, v, logN, tile, tw);
#pragma unroll
    for (u32 j = 0; j < TL::R; ++j) {                              // a thread's own slots
        if (RD + 1 < TL::ROUNDS) {
            lds[RN::slot(j)] = f.bits(v[j]);
        } else if (RAW) {
            f.norm(v[j]);
            lds[RN::slot(j)] = f.bits(v[j]);
        } else {
            lds[RN::slot(j)] = f.out(v[j]);
        }
    }
    exchange_sync<RN::BEHIND>();
    if constexpr (RD + 1 < TL::ROUNDS) fwd_rounds<RAW, RL, RD + 1>(f, logN, tile, lds, next);
}

// forward: load(idx) gives the residue at index idx of the polynomial, as the first pass has left it (N = 2^12: canonical; first
// round's pattern: coalesced); on
// return the tile's transformed, canonical residues are in LDS, where a thread may read what Tile::one or Tile::pair give
// it (RL = 4: the workgroup is synced).  RAW: the residues are
// left in the field's own form instead (f.bits of a value brought back by f.norm: for the fp64 field a double with
// |x| <= q/2), for a caller that goes on computing in that field and would only convert them back.
// FIELD: raw holds the field's own values whatever the ring.
template <bool RAW = false, u32 RL = 4, bool FIELD = false, class F>
__device__ __forceinline__ void pass_b_fwd_from_regs(const F &f, u32 logN, u64 *lds, const u64 (&raw)[1u << RL], u32 tile) {
    typedef Tile<RL> TL;
    typedef Round<RL, 0> RN;
    Twids<RL, 0, F> tw;
    Twids<RL, 1, F> next;
    load_twids<RL, 0>(f, logN, tile, tw);
    typename F::T v[TL::R];
    if (!FIELD && logN == 12) {
#pragma unroll
        for (u32 j = 0; j < TL::R; ++j) v[j] = f.in(raw[j]);
    } else {
#pragma unroll
        for (u32 j = 0; j < TL::R; ++j) v[j] = f.from_bits(raw[j]);
    }
    load_twids<RL, 1>(f, logN, tile, next);
    round_fwd<RL, 0>(f, v, logN, tile, tw);
#pragma unroll
    for (u32 j = 0; j < TL::R; ++j) lds[RN::slot(j)] = f.bits(v[j]);
    exchange_sync<RN::BEHIND>();
    fwd_rounds<RAW, RL, 1>(f, logN, tile, lds, next);
}
template <bool RAW = false, u32 RL = 4, class F, class Load>
__device__ __forceinline__ void pass_b_fwd_to_lds(const F &f, u32 logN, u64 *lds, Load load) {
    u64 raw[1u << RL];
#pragma unroll
    for (u32 j = 0; j < (1u << RL); ++j) raw[j] = load((blockIdx.x << 12) + Round<RL, 0>::elem(j));
    pass_b_fwd_from_regs<RAW, RL>(f, logN, lds, raw, blockIdx.x);
}

// inverse rounds from RD down to the second, LDS to LDS; the residues in front of the first of them are canonical
template <u32 RL, u32 RD, class F>
__device__ __forceinline__ void inv_rounds(const F &f, u32 logN, u64 *lds, const Twids<RL, RD, F> &tw, Twids<RL, 0, F> &tw0) {
    typedef Tile<RL> TL;
    typedef Round<RL, RD> RN;
    Twids<RL, RD - 1, F> next;
    load_twids<RL, RD - 1>(f, logN, blockIdx.x, next);
    typename F::T v[TL::R];
#pragma unroll
    for (u32 j = 0; j < TL::R; ++j) {
        const u64 x = lds[RN::slot(j)];
        v[j] = RD + 1 == TL::ROUNDS ? f.in(x) : f.from_bits(x);
    }
    round_inv<RL, RD>(f, v, logN, blockIdx.x, tw, false);
#pragma unroll
    for (u32 j = 0; j < TL::R; ++j) lds[RN::slot(j)] = f.bits(v[j]);   // a thread's own slots
    exchange_sync<RN::FRONT>();
    if constexpr (RD > 1)
        inv_rounds<RL, RD - 1>(f, logN, lds, next, tw0);
    else
        tw0 = next;
}

// inverse: expects the tile's canonical residues in LDS, written in the pattern of Tile::one or Tile::pair (the exchange
// itself is synced here);
// store(idx, value) receives the results in the first round's pattern (coalesced), for the other pass to go on with.  A tile that is the whole
// polynomial (N = 2^12) ends the transform in the last round, which folds in N^-1.
template <u32 RL = 4, class F, class Store>
__device__ __forceinline__ void pass_b_inv_from_lds(const F &f, u32 logN, u64 *lds, Store store) {
    typedef Tile<RL> TL;
    typedef Round<RL, 0> RN;
    const u32 base = blockIdx.x << 12;
    Twids<RL, TL::ROUNDS - 1, F> tw;
    Twids<RL, 0, F> tw0;
    load_twids<RL, TL::ROUNDS - 1>(f, logN, blockIdx.x, tw);
    exchange_sync<TL::WAVE ? 64 : TL::THREADS>();
    inv_rounds<RL, TL::ROUNDS - 1>(f, logN, lds, tw, tw0);
    typename F::T v[TL::R];
#pragma unroll
    for (u32 j = 0; j < TL::R; ++j) v[j] = f.from_bits(lds[RN::slot(j)]);
    round_inv<RL, 0>(f, v, logN, blockIdx.x, tw0, logN == 12);
    if (logN == 12) {                                                // one branch: not one per residue
#pragma unroll
        for (u32 j = 0; j < TL::R; ++j) store(base + RN::elem(j), f.out(v[j]));
    } else {
#pragma unroll
        for (u32 j = 0; j < TL::R; ++j) store(base + RN::elem(j), f.half(v[j]));
    }
}

// Whole pass with coalesced stores (forward) / coalesced loads (inverse).
template <bool INV, u32 RL = 4, class F, class Load, class Store>
__device__ __forceinline__ void pass_b_body(const F &f, u32 logN, u64 *lds, Load load, Store store) {
    typedef Tile<RL> TL;
    const u32 tid = threadIdx.x, base = blockIdx.x << 12;
    if (!INV) {
        pass_b_fwd_to_lds<false, RL>(f, logN, lds, load);
#pragma unroll
        for (u32 i = 0; i < TL::R; ++i) store(base + TL::one(tid, i), lds[TL::slot(TL::one(tid, i))]);
    } else {
#pragma unroll
        for (u32 i = 0; i < TL::R; ++i) lds[TL::slot(TL::one(tid, i))] = load(base + TL::one(tid, i));
        pass_b_inv_from_lds<RL>(f, logN, lds, store);
    }
}

// A row of residues behind a buffer descriptor: entry at + col, at the same for the wavefront.  The address of an access is one
// scalar and one vector register; as pointers, sixteen rows of a column take 32 vector registers, computed ahead of the pass.
struct RowBuf {
    typedef u32 u32x2 __attribute__((ext_vector_type(2)));
    __amdgpu_buffer_rsrc_t rs;
    __device__ __forceinline__ RowBuf(const u64 *row, u32 n)
        : rs(__builtin_amdgcn_make_buffer_rsrc(const_cast<u64 *>(row), 0, (int)(n * sizeof(u64)), 0x00020000)) {}
    __device__ __forceinline__ u64 load(u32 at, u32 col) const {
        return __builtin_bit_cast(u64, __builtin_amdgcn_raw_buffer_load_b64(rs, (int)(col * 8), (int)(at * 8), 0));
    }
    template <bool NT = false>
    __device__ __forceinline__ void store(u32 at, u32 col, u64 v) const {
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), rs, (int)(col * 8), (int)(at * 8), NT ? 2 : 0);
    }
};

// pass A for N = 2^(12+LOGR), LOGR > 0: the first LOGR stages pair residues 4096 apart, so a thread that owns one of the 4096
// columns holds its 2^LOGR rows in registers: no LDS, every access a run of consecutive residues.  col: the thread's
// column; load(at, col) / store(at, col, value) see residues at index at + col of the polynomial, canonical on the side of
// the coefficients, at the same for all threads: a scalar address to which a thread adds one 32-bit offset (an address per
// row would take 32 registers).
template <bool INV, u32 LOGR, class F, class Load, class Store>
__device__ __forceinline__ void pass_a_body(const F &f, u32 col, Load load, Store store) {
    static_assert(LOGR > 0, "at N = 2^12 the tile pass is the whole transform");
    constexpr u32 R = 1u << LOGR;
    typename F::T v[R];
#pragma unroll
    for (u32 j = 0; j < R; ++j) v[j] = INV ? f.from_bits(load(j * 4096, col)) : f.in(load(j * 4096, col));
    if constexpr (INV)
        radix_inv<LOGR, true, false>(f, v, 0, 0, true);
    else
        radix_fwd<LOGR>(f, v, 0, 0);
#pragma unroll
    for (u32 j = 0; j < R; ++j) store(j * 4096, col, INV ? f.out(v[j]) : f.half(v[j]));
}

// Field objects for limb `limb` from the parameter tables.
__device__ __forceinline__ FieldFp make_field_fp(const ModFp &mf, const double *twf, u32 limb, u32 logN) {
    FieldFp f;
    f.q = mf.q;
    f.u = mf.u;
    f.n0 = mf.ninv;
    f.n1 = mf.ninv_w;
    f.tw = twf + ((size_t)limb << logN);
    return f;
}

// tws: [W][N][2]: four words of 32 bits per twiddle, ninvs [W][4]: two such, N^-1 and N^-1 psi^-(N/2)
__device__ __forceinline__ TwPm<true> pm_words(const u64 *p) {
    return TwPm<true>{(int)p[0], (int)(p[0] >> 32), (int)p[1], (int)(p[1] >> 32)};
}
__device__ __forceinline__ FieldPm make_field_pm(const ModConst *mods, const u64 *tws, const u64 *ninvs, u32 limb, u32 logN) {
    FieldPm f;
    f.q = mods[limb].q;
    f.q8 = 8 * f.q;
    const u32 b = 64 - __builtin_clzll(f.q);
    f.s = b - 32;
    f.p2s = 1u << f.s;
    f.c = (int)(((u64)1 << b) - f.q);
    f.r31 = (int64_t)1 << 31;
    f.mid = -((int64_t)1 << (b - 1));
    asm("" : "+v"(f.r31), "+v"(f.mid));             // kept in vector registers: an instruction reads one scalar operand
    f.tw = reinterpret_cast<const int4 *>(tws) + ((size_t)limb << logN);
    f.n0 = pm_words(ninvs + 4 * limb);
    f.n1 = pm_words(ninvs + 4 * limb + 2);
    return f;
}

// tws: [W][N] pairs (w, w') as consecutive words, ninvs: [W][4] = N^-1, its quotient, N^-1 psi^-(N/2), its quotient
__device__ __forceinline__ FieldInt make_field_int(const ModConst *mods, const u64 *tws, const u64 *ninvs, u32 limb,
                                                   u32 logN) {
    FieldInt f;
    f.q = mods[limb].q;
    f.q2 = 2 * f.q;
    f.tw = reinterpret_cast<const ulonglong2 *>(tws) + ((size_t)limb << logN);
    f.n0 = TwInt{ninvs[4 * limb], ninvs[4 * limb + 1]};
    f.n1 = TwInt{ninvs[4 * limb + 2], ninvs[4 * limb + 3]};
    return f;
}

// body(field of the limb); with_int_field: of a limb that is known to be 2^50 or more
template <class Body>
__device__ __forceinline__ void with_int_field(const ModFp &mf, const ModConst *mods, const u64 *tws, const u64 *ninvs,
                                               u32 limb, u32 logN, Body body) {
    if (mf.pm)
        body(make_field_pm(mods, tws, ninvs, limb, logN));
    else
        body(make_field_int(mods, tws, ninvs, limb, logN));
}
template <class Body>
__device__ __forceinline__ void with_field(const ModFp &mf, const ModConst *mods, const u64 *tws, const double *twf,
                                           const u64 *ninvs, u32 limb, u32 logN, Body body) {
    if (mf.ok)
        body(make_field_fp(mf, twf, limb, logN));
    else
        with_int_field(mf, mods, tws, ninvs, limb, logN, body);
}

}  // namespace ckks
