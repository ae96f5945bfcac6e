// Complex-slot encode / decode on the device (Sec. 2.1 Encode / Decode, Sec. 3.1 slot order).
// Slot j of a plaintext m(X) is m(zeta^(5^j)), zeta = exp(i*pi/N).
//
// Decode.  With w_k = m_k + i*m_(k+n), k < n = N/2, zeta^(5^j n) = i gives z_j = sum_k w_k zeta^(5^j k): n complex values
// in, n out.  Since 5^(n/2) = 1 + N (mod 2N), the sum splits into the even and the odd k like an FFT,
//   z_j, z_(j+n/2) = E_j +- zeta^(5^j) O_j,   j < n/2,
// with E, O the same transform at half the length.  The butterflies run from length 2 up to n on w in bit-reversed order;
// the slots come out in order, and the twiddle of butterfly j of half length h is tw[h + j] = exp(2*pi*i*(5^j mod 8h)/(8h)).
//
// Encode.  With e_j = 5^j mod 2N and bin t_j = (e_j - 1)/2,
//   m_k = (1/N) * Re( zeta^(-k) * sum_t v_t * exp(-2*pi*i*t*k/N) ),  v[t_j] = z_j,  v[N-1-t_j] = conj(z_j):
// an N-point FFT, decimation in frequency with the twiddles w[j << s] of a table of N-th roots, and a twist.  (The
// half-length form of decode would do for encode too, but rounds differently: an encoded integer next to a tie could
// change by one, and with it every residue of a weight or message that a program encodes again.  These are the operations
// of a plain radix-2 FFT in their order, so the integers are the same whatever the passes are.)
//
// Two passes over 4096-element tiles each, 16 elements per thread and at most four stages (radix 16) between exchanges
// through LDS in decode, 8 and three in encode:
//   far:  the stages of half length 256 and more, on columns (elements 256 apart); slots on one side, scratch on the other.
//   near: the stages of half length up to 128, on 16 runs of 256 elements that lie a sixteenth of the array apart: then the
//         tile's k = bitrev(p) form runs of 16, a 128-byte line of the coefficients on the other side.
// Encode's far pass finds its columns by their slots: t_j mod 256 depends on j mod 128 alone, so the columns of COLS/2
// neighbouring j mod 128 are read from whole lines of slots, and the columns 255 - (t mod 256) are their conjugates.  It
// leaves column (group, member) at place group * COLS + member of the scratch rows, and reads twiddles laid out by place:
// by column, each lane's lies in a cache line of its own, and the pass waits for the lines (96 vectors at N = 2^16: the two
// launches 50.6 us, 37.6 so).
// A pass reads and writes every element once, and nothing else touches memory.  Short rings: one workgroup per vector.
// Off the server's hot path.  96 real vectors at N = 2^16: 308 us with permutation, transform, twist and rounding in
// five kernels, 75 us now (0.3 GB past the caches: 60 at the rate of a copy); 5 vectors decoded at N = 2^15: 45 us, 12 us now.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "ckks_internal.h"
#include "common_kernels.h"
#include "mac_device.h"
#include "ntt_device.h"

namespace ckks {

constexpr u32 FFT_TILE = 4096;
// Threads of a workgroup.  Two tiles fit a CU's LDS, so a wavefront count per SIMD of 2 with 16 elements per thread and of 4
// with 8, for one exchange more (3 + 3 + 2 stages instead of 4 + 4).  Encode, us, 16 and 8 elements per thread: 1 / 40 / 200
// vectors at 2^13 12.3 / 14.5 / 63 and 10.6 / 13.0 / 56, 4 / 96 at 2^15 14.1 / 58.0 and 13.1 / 55.5, 16 / 200 at 2^16
// 28.5 / 210 and 25.4 / 191.  Decode's far pass gains nothing by it: 1 / 5 / 64 vectors at 2^15 10.9 / 12.0 / 22.3 and
// 11.2 / 12.1 / 22.9, 200 at 2^16 132 and 131.
constexpr u32 FFT_THREADS = 256, ENC_THREADS = 512;
constexpr u32 ENC_CHUNK = 64;         // vectors transformed per scratch chunk (N = 2^16: 64 MiB for encode)
// tile element i: one pad element after 16 and one after 256, so that runs of 16, strides of 16 and strides of 256 all
// fall on distinct banks.  70 KB: two workgroups per CU.
__device__ __forceinline__ u32 fft_slot(u32 i) { return i + (i >> 4) + (i >> 8); }
constexpr u32 FFT_LDS = FFT_TILE + FFT_TILE / 16 + FFT_TILE / 256;

__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
    return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ double2 cadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ double2 csub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }

// The same with two roundings per component instead of three.  Decode takes this: its twiddles have no zeros and ones among
// them as those of an N-point transform have, and with plain products its slots were 1.4 to 2.4 % further (rms) from exact
// ones than an N-point radix-2 transform's on rings from 2^10 to 2^16; with these they are 3.4 to 4.4 % nearer.  (Products
// that also recover the first one's rounding: 4.4 to 5.1 %, and 70 vectors at 2^16 1.5 % slower than with plain ones.)
// Encode keeps plain products: an integer next to a tie may not move.
__device__ __forceinline__ double2 cmul_fma(double2 a, double2 b) {
    return make_double2(fma(a.x, b.x, -(a.y * b.y)), fma(a.x, b.y, a.y * b.x));
}

// LOGR stages on elements off + r * stride, r < 2^LOGR, of every block of 2^LOGR * stride.  Encode: half lengths
// stride << (LOGR-1) down to stride, (a + b, (a - b) w); decode: the other way round, (a + b w, a - b w).
template <u32 LOGR, bool ENC>
__device__ __forceinline__ void fft_group(double2 *v, const double2 *__restrict__ tw, u32 stride, u32 off) {
    constexpr u32 R = 1u << LOGR;
#pragma unroll
    for (u32 s = 0; s < LOGR; ++s) {
        const u32 t = ENC ? s : LOGR - 1 - s, g = R >> (t + 1);
#pragma unroll
        for (u32 i = 0; i < g; ++i) {
            const double2 w = tw[(g + i) * stride + off];
#pragma unroll
            for (u32 k = 0; k < (1u << t); ++k) {
                double2 &a = v[k * 2 * g + i], &b = v[k * 2 * g + i + g];
                const double2 x = a, y = ENC ? b : cmul_fma(b, w);
                a = cadd(x, y);
                b = ENC ? cmul(csub(x, y), w) : csub(x, y);
            }
        }
    }
}

// Where the coefficients meet the transform of encode: X_k into the caller's array.
struct EncodeOut {
    int64_t *c;                // the vector's N coefficients
    const double2 *twist;      // [N]: zeta^(-k)
    u32 N, real;
    double mul;
    // Coefficient k = nearest integer to (scale/N) * Re(zeta^(-k) * X_k).  A real slot vector is fixed by conjugation, so
    // its polynomial satisfies m[N-k] = -m[k] and m[N/2] = 0 exactly; real != 0 imposes that on the rounded values (the
    // transform gives it only up to rounding) and takes k < N/2 alone.
    __device__ __forceinline__ void put(u32 k, double2 x) const {
        const double2 t = twist[k];
        const int64_t v = (int64_t)rint((x.x * t.x - x.y * t.y) * mul);
        c[k] = v;
        if (real) c[k ? N - k : N / 2] = k ? -v : 0;
    }
};

struct DecodeIn {
    const u64 *r;              // the vector's residues [nlimbs][N]
    u32 n, nlimbs;
    u64 q0, q1, q0inv_mont;
    ModConst m1;
    double q0inv, uq;          // two primes below 2^50: q0^-1 mod q1 and 1/q1; otherwise 0
    // centred lift of the residues on one or two primes
    __device__ __forceinline__ double lift(u64 r0, u64 r1) const {
        if (q0inv != 0.0) {
            // x = r0 + q0 * t with t = (r1 - r0) * q0^-1 mod q1 the representative in [-(q1-1)/2, (q1-1)/2], every step
            // an exact integer in doubles up to the last, one rounding.  x <= Q/2 fails for t = (q1-1)/2 with r0 > q0/2
            // alone.  (A lift in 128-bit integers takes about ten times the instructions, which is what a decode of a few
            // vectors waits for: 5 vectors at N = 2^15 21.3 us, 16.3 us with this.)
            const double q = (double)q1, hq = (double)(q1 >> 1), a = canonical_double(r0), d = canonical_double(r1) - a;
            const double h = d * q0inv, l = fma(d, q0inv, -h);
            double t = fma(-rint(h * uq), q, h) + l;
            if (t > hq) t -= q;
            if (t < -hq) t += q;
            if (t == hq && r0 > q0 / 2) t -= q;
            return fma(t, (double)q0, a);
        }
        if (nlimbs == 1) return r0 > q0 / 2 ? -(double)(q0 - r0) : (double)r0;
        // x = r0 + q0 * ((r1 - r0) * q0^-1 mod q1), then centred modulo q0*q1
        // (mont_mul takes any 64-bit first factor: no division for r0 mod q1)
        const u64 t = sub_mod(mont_mul(r1, q0inv_mont, m1), mont_mul(r0, q0inv_mont, m1), q1);
        const unsigned __int128 Q = (unsigned __int128)q0 * q1;
        unsigned __int128 y = (unsigned __int128)q0 * t + r0;
        const bool neg = y > Q / 2;
        if (neg) y = Q - y;
        const double x = (double)(u64)(y >> 64) * 18446744073709551616.0 + (double)(u64)y;
        return neg ? -x : x;
    }
    struct Raw {
        u64 a0, a1, b0, b1;    // coefficients k and n + k on the two primes
    };
    __device__ __forceinline__ Raw load(u32 k) const {
        const u32 two = nlimbs == 1 ? 0 : 2 * n;
        return Raw{r[k], r[two + k], r[n + k], r[two + n + k]};
    }
    __device__ __forceinline__ double2 get(const Raw &w) const { return make_double2(lift(w.a0, w.a1), lift(w.b0, w.b1)); }
};

// Workgroup -> tile x of vector y.  Workgroups go to the XCDs round-robin, each of which has its own L2: every eight vectors
// are dealt to the eight, all tiles of one to the same, which find each other's lines of slots and scratch there and complete
// each other's lines of coefficients (a mirrored run k -> N - k crosses lines).  Encode without and with, us: 40 / 96 / 200 general
// vectors at 2^14 17.2 / 37.5 / 75.7 and 13.8 / 30.3 / 63.0, at 2^15 28.9 / 51.5 / 107 and 23.7 / 48.0 / 94.8, 16 / 96 at
// 2^16 22.7 / 78.2 and 20.4 / 77.8; 2^17 the same, 2^13 too (8 to 400 vectors, two tiles each: within 1 %).  Decode, for eight vectors and more at 2^14 to
// 2^16: 64 vectors at 2^14 15.9 and 13.6, 40 at 2^15 17.9 and 14.6, 16 / 200 at 2^16 18.4 / 104 and 13.8 / 100; at 2^13, where
// a vector is one tile, and for fewer vectors the step costs 1 to 3 %, at 2^17 it gives 20 % of 16 and takes 2 % of 40.  The
// vectors after the last eight: in order.
__device__ __forceinline__ void deal_vectors(u32 &x, u32 &y) {
    if (y >= (gridDim.y & ~7u)) return;
    const u32 lin = y * gridDim.x + x, slot = lin >> 3;
    y = uniform_div(slot, gridDim.x);
    x = slot - y * gridDim.x;
    y = y * 8 + (lin & 7);
}

// Far pass of decode: scratch -> slots, times inv_scale.  n = 256 << S.
// grid: x = group of 4096 >> S columns, y = vector
template <u32 S, bool DEAL>
__global__ __launch_bounds__(FFT_THREADS) void decode_far_kernel(const double2 *__restrict__ in, double2 *__restrict__ out,
                                                                 const double2 *__restrict__ tw, double inv_scale) {
    constexpr u32 COLS = FFT_TILE >> S, LOW = S - 4, SUB = 1u << LOW, n = 256u << S;
    __shared__ double2 tile[FFT_LDS];
    u32 grp = blockIdx.x, vec = blockIdx.y;
    if (DEAL) deal_vectors(grp, vec);
    const u32 col = threadIdx.x % COLS, q = threadIdx.x / COLS;              // q < SUB
    const u32 pcol = grp * COLS + col;
    const double2 *src = in + (size_t)vec * n + pcol;
    double2 *dst = out + (size_t)vec * n + pcol;
    double2 v[16];
    // rows (q + SUB * m) * SUB + r, r < SUB: the low row bits; rows r * SUB + q: the top four
    auto low_row = [&](u32 e) { return (q + SUB * (e >> LOW)) * SUB + (e & (SUB - 1)); };
    auto top_row = [&](u32 r) { return r * SUB + q; };
#pragma unroll
    for (u32 e = 0; e < 16; ++e) v[e] = src[low_row(e) * 256];
    if constexpr (LOW > 0) {
#pragma unroll
        for (u32 m = 0; m < (16u >> LOW); ++m) fft_group<LOW, false>(v + m * SUB, tw, 256, pcol);
#pragma unroll
        for (u32 e = 0; e < 16; ++e) tile[fft_slot(low_row(e) * COLS + col)] = v[e];
        __syncthreads();
#pragma unroll
        for (u32 r = 0; r < 16; ++r) v[r] = tile[fft_slot(top_row(r) * COLS + col)];
    }
    fft_group<4, false>(v, tw, SUB * 256, q * 256 + pcol);
#pragma unroll
    for (u32 r = 0; r < 16; ++r) dst[top_row(r) * 256] = make_double2(v[r].x * inv_scale, v[r].y * inv_scale);
}

// Near pass of decode: residues -> scratch.  grid: x = n / 4096, y = vector
template <bool DEAL>
__global__ __launch_bounds__(FFT_THREADS) void decode_near_kernel(double2 *__restrict__ scratch,
                                                                  const double2 *__restrict__ tw, DecodeIn coef,
                                                                  size_t coef_stride, u32 logn) {
    __shared__ double2 tile[FFT_LDS];
    const u32 tid = threadIdx.x, h = tid >> 4, c = tid & 15, fb = logn - 12;
    u32 f = blockIdx.x, vec = blockIdx.y;
    if (DEAL) deal_vectors(f, vec);
    double2 *v0 = scratch + ((size_t)vec << logn) + (((h << fb) + f) << 8);     // run h of the tile
    coef.r += vec * coef_stride;
    // coefficient side: thread (m & 15 = h, hh = c) holds element lo = bitrev8(m) of run bitrev4(hh), k as below
    const u32 ch = __brev(c) >> 28, fk = (fb ? __brev(f) >> (32 - fb) : 0) * 16 + c;
    auto side = [&](u32 r) { return fft_slot(ch * 256 + (__brev(h + 16 * r) >> 24)); };
    auto kidx = [&](u32 r) { return ((h + 16 * r) << (logn - 8)) + fk; };
    double2 v[16];
#pragma unroll
    for (u32 r0 = 0; r0 < 16; r0 += 8) {               // the loads of eight coefficients are in flight together
        DecodeIn::Raw w[8];
#pragma unroll
        for (u32 r = 0; r < 8; ++r) w[r] = coef.load(kidx(r0 + r));
#pragma unroll
        for (u32 r = 0; r < 8; ++r) tile[side(r0 + r)] = coef.get(w[r]);
    }
    __syncthreads();
#pragma unroll
    for (u32 r = 0; r < 16; ++r) v[r] = tile[fft_slot(h * 256 + c * 16 + r)];
    fft_group<4, false>(v, tw, 1, 0);
#pragma unroll
    for (u32 r = 0; r < 16; ++r) tile[fft_slot(h * 256 + c * 16 + r)] = v[r];          // a thread's own slots
    __syncthreads();
#pragma unroll
    for (u32 r = 0; r < 16; ++r) v[r] = tile[fft_slot(h * 256 + c + 16 * r)];
    fft_group<4, false>(v, tw, 16, c);
#pragma unroll
    for (u32 r = 0; r < 16; ++r) v0[c + 16 * r] = v[r];
}

// The same by 1024 threads with four elements each: the same operations on the same values, two stages at a time instead of
// four, with all of a thread's coefficients and twiddles on their way at once and, a run belonging to one wavefront, no
// barrier behind the first exchange.
template <bool DEAL>
__global__ __launch_bounds__(1024) void decode_near_wide_kernel(double2 *__restrict__ scratch, const double2 *__restrict__ tw,
                                                                DecodeIn coef, size_t coef_stride, u32 logn) {
    __shared__ double2 tile[FFT_LDS];
    const u32 tid = threadIdx.x, fb = logn - 12;
    u32 f = blockIdx.x, vec = blockIdx.y;
    if (DEAL) deal_vectors(f, vec);
    coef.r += vec * coef_stride;
    {
        const u32 h = tid >> 4, c = tid & 15, ch = __brev(c) >> 28, fk = (fb ? __brev(f) >> (32 - fb) : 0) * 16 + c;
        DecodeIn::Raw w[4];
#pragma unroll
        for (u32 r = 0; r < 4; ++r) w[r] = coef.load(((h + 64 * r) << (logn - 8)) + fk);
#pragma unroll
        for (u32 r = 0; r < 4; ++r) tile[fft_slot(ch * 256 + (__brev(h + 64 * r) >> 24))] = coef.get(w[r]);
    }
    const u32 run = tid >> 6, lane = tid & 63;
    double2 *v0 = scratch + ((size_t)vec << logn) + (((run << fb) + f) << 8);
    double2 w[4][3];                                               // of the halves 4^k and 2 4^k
#pragma unroll
    for (u32 k = 0; k < 4; ++k) {
        const u32 stride = 1u << (2 * k), off = lane & (stride - 1);
        w[k][0] = tw[stride + off];
        w[k][1] = tw[2 * stride + off];
        w[k][2] = tw[3 * stride + off];
    }
    __syncthreads();
#pragma unroll
    for (u32 k = 0; k < 4; ++k) {
        const u32 stride = 1u << (2 * k), first = (lane >> (2 * k) << (2 * k + 2)) + (lane & (stride - 1));
        double2 v[4];
#pragma unroll
        for (u32 r = 0; r < 4; ++r) v[r] = tile[fft_slot(run * 256 + first + r * stride)];
#pragma unroll
        for (u32 s = 0; s < 2; ++s)
#pragma unroll
            for (u32 i = 0; i < 2; ++i) {
                double2 &a = v[s ? i : 2 * i], &b = v[s ? i + 2 : 2 * i + 1];
                const double2 x = a, y = cmul_fma(b, w[k][s ? 1 + i : 0]);
                a = cadd(x, y);
                b = csub(x, y);
            }
        if (k < 3) {
#pragma unroll
            for (u32 r = 0; r < 4; ++r) tile[fft_slot(run * 256 + first + r * stride)] = v[r];   // a thread's own slots
            exchange_sync<64>();
        } else {
#pragma unroll
            for (u32 r = 0; r < 4; ++r) v0[first + r * stride] = v[r];
        }
    }
}

// n < 4096: the whole decode of one vector in LDS, one exchange per stage.  grid: x = vector
__global__ __launch_bounds__(FFT_THREADS) void decode_small_kernel(double2 *__restrict__ out,
                                                                   const double2 *__restrict__ tw, DecodeIn coef,
                                                                   size_t coef_stride, u32 logn, double inv_scale) {
    __shared__ double2 tile[FFT_TILE / 2];
    const u32 n = 1u << logn;
    coef.r += blockIdx.x * coef_stride;
    for (u32 i = threadIdx.x; i < n; i += FFT_THREADS) tile[i] = coef.get(coef.load(__brev(i) >> (32 - logn)));
    __syncthreads();
    for (u32 lh = 0; lh < logn; ++lh) {
        const u32 half = 1u << lh;
        for (u32 b = threadIdx.x; b < n / 2; b += FFT_THREADS) {
            const u32 j = b & (half - 1), i0 = ((b >> lh) << (lh + 1)) + j, i1 = i0 + half;
            const double2 x = tile[i0], y = cmul_fma(tile[i1], tw[half + j]);
            tile[i0] = cadd(x, y);
            tile[i1] = csub(x, y);
        }
        __syncthreads();
    }
    for (u32 i = threadIdx.x; i < n; i += FFT_THREADS)
        out[(size_t)blockIdx.x * n + i] = make_double2(tile[i].x * inv_scale, tile[i].y * inv_scale);
}

// Far pass of encode: slots -> scratch (columns in the order of their slots).  N = 256 << S rows of 256.
// bin[j] = t_j.  grid: x = group of 4096 >> S columns, y = vector
template <u32 S>
__global__ __launch_bounds__(ENC_THREADS, 4) void encode_far_kernel(const double2 *__restrict__ slots,
                                                                 double2 *__restrict__ out,
                                                                 const double2 *__restrict__ tw,
                                                                 const u32 *__restrict__ bin, u32 real) {
    constexpr u32 COLS = FFT_TILE >> S, SC = COLS / 2, ROWS = 1u << S, N = 256u << S, TPC = ROWS / 8;
    __shared__ double2 tile[FFT_LDS];
    u32 grp = blockIdx.x, vec = blockIdx.y;
    deal_vectors(grp, vec);
    const double2 *src = slots + (size_t)vec * (N / 2) + grp * SC;
#pragma unroll
    for (u32 l = 0; l < FFT_TILE / 2 / ENC_THREADS; ++l) {
        const u32 idx = threadIdx.x + ENC_THREADS * l, x = idx % SC, j = x + 128 * (idx / SC);
        double2 z = src[j];
        if (real) z.y = 0.0;
        const u32 row = bin[grp * SC + j] >> 8;
        tile[fft_slot(row * COLS + x)] = z;
        tile[fft_slot((ROWS - 1 - row) * COLS + SC + x)] = make_double2(z.x, -z.y);
    }
    __syncthreads();
    const u32 col = threadIdx.x % COLS, q = threadIdx.x / COLS;              // q < TPC
    const u32 place = grp * COLS + col;                                      // as the twiddles lie
    double2 *dst = out + (size_t)vec * N + place;
    // G stages on row bits B0 .. B0+G-1: a thread takes 8 >> G of the 2^(S-G) combinations of the other row bits
    auto group = [&](auto b0, auto g) {
        constexpr u32 B0 = decltype(b0)::value, G = decltype(g)::value, R = 1u << G;
        double2 v[8];
        auto row = [&](u32 m, u32 r) {
            const u32 o = q + TPC * m;
            return ((o >> B0) << (B0 + G)) + (r << B0) + (o & ((1u << B0) - 1));
        };
#pragma unroll
        for (u32 m = 0; m < (8u >> G); ++m) {
#pragma unroll
            for (u32 r = 0; r < R; ++r) v[m * R + r] = tile[fft_slot(row(m, r) * COLS + col)];
            fft_group<G, true>(v + m * R, tw, 256u << B0, ((q + TPC * m) & ((1u << B0) - 1)) * 256 + place);
        }
#pragma unroll
        for (u32 m = 0; m < (8u >> G); ++m)
#pragma unroll
            for (u32 r = 0; r < R; ++r) {
                if (B0 == 0)
                    dst[row(m, r) * 256] = v[m * R + r];
                else
                    tile[fft_slot(row(m, r) * COLS + col)] = v[m * R + r];                 // a thread's own slots
            }
        if (B0 != 0) __syncthreads();
    };
    using std::integral_constant;
    group(integral_constant<u32, S - 3>(), integral_constant<u32, 3>());
    if constexpr (S > 6) {
        group(integral_constant<u32, S - 6>(), integral_constant<u32, 3>());
        group(integral_constant<u32, 0>(), integral_constant<u32, S - 6>());
    } else {
        group(integral_constant<u32, 0>(), integral_constant<u32, S - 3>());
    }
}

// Near pass of encode: scratch -> coefficients.  colmap[place] = the column at that place of a scratch row.
// grid: x = N / 4096, y = vector
__global__ __launch_bounds__(ENC_THREADS, 4) void encode_near_kernel(const double2 *__restrict__ scratch,
                                                                     const double2 *__restrict__ tw,
                                                                     const u32 *__restrict__ colmap, EncodeOut coef,
                                                                     u32 logN) {
    __shared__ double2 tile[FFT_LDS];
    const u32 tid = threadIdx.x, fb = logN - 12;
    u32 f = blockIdx.x, vec = blockIdx.y;
    deal_vectors(f, vec);
    coef.c += (size_t)vec << logN;
    double2 v[8];
    {
        const u32 place = tid & 255, odd = tid >> 8, lo = colmap[place];
        const double2 *v0 = scratch + ((size_t)vec << logN) + (f << 8) + place;
#pragma unroll
        for (u32 r = 0; r < 8; ++r) v[r] = v0[(size_t)(2 * r + odd) << (fb + 8)];      // run 2r + odd
#pragma unroll
        for (u32 r = 0; r < 8; ++r) tile[fft_slot((2 * r + odd) * 256 + lo)] = v[r];
    }
    __syncthreads();
    const u32 run = tid >> 5 << 8, c = tid & 31;                                       // half a wavefront per run
    // 3, 3 and 2 of the 8 stages
    auto first = [&](u32 r) { return fft_slot(run + c + 32 * r); };
    auto second = [&](u32 r) { return fft_slot(run + (c >> 2) * 32 + (c & 3) + 4 * r); };
    auto third = [&](u32 r) { return fft_slot(run + c * 8 + r); };
#pragma unroll
    for (u32 r = 0; r < 8; ++r) v[r] = tile[first(r)];
    fft_group<3, true>(v, tw, 32, c);
#pragma unroll
    for (u32 r = 0; r < 8; ++r) tile[first(r)] = v[r];                                 // a thread's own slots
    exchange_sync<64>();
#pragma unroll
    for (u32 r = 0; r < 8; ++r) v[r] = tile[second(r)];
    fft_group<3, true>(v, tw, 4, c & 3);
#pragma unroll
    for (u32 r = 0; r < 8; ++r) tile[second(r)] = v[r];                                // a thread's own slots
    exchange_sync<64>();
#pragma unroll
    for (u32 r = 0; r < 8; ++r) v[r] = tile[third(r)];
    fft_group<2, true>(v, tw, 1, 0);
    fft_group<2, true>(v + 4, tw, 1, 0);
#pragma unroll
    for (u32 r = 0; r < 8; ++r) tile[third(r)] = v[r];                                 // a thread's own slots
    __syncthreads();
    // thread (m & 31, hh = low bits) writes k = m 2^(logN-8) + ..., element lo = bitrev8(m) of run bitrev4(hh)
    const u32 h = tid >> 4, hh = tid & 15, ch = __brev(hh) >> 28, fk = (fb ? __brev(f) >> (32 - fb) : 0) * 16 + hh;
#pragma unroll
    for (u32 r = 0; r < 8; ++r) {
        const u32 m = h + 32 * r;
        if (coef.real && r >= 4) break;                                                // k >= N/2
        coef.put((m << (logN - 8)) + fk, tile[fft_slot(ch * 256 + (__brev(m) >> 24))]);
    }
}

// N <= 4096: the whole encode of one vector in LDS, one exchange per stage.  grid: x = vector
__global__ __launch_bounds__(FFT_THREADS) void encode_small_kernel(const double2 *__restrict__ slots,
                                                                   const double2 *__restrict__ tw,
                                                                   const u32 *__restrict__ bin, EncodeOut coef,
                                                                   u32 logN, u32 real) {
    __shared__ double2 tile[FFT_TILE];
    const u32 N = 1u << logN, n = N / 2;
    coef.c += (size_t)blockIdx.x << logN;
    for (u32 j = threadIdx.x; j < n; j += FFT_THREADS) {
        double2 z = slots[(size_t)blockIdx.x * n + j];
        if (real) z.y = 0.0;
        const u32 t = bin[j];
        tile[t] = z;
        tile[N - 1 - t] = make_double2(z.x, -z.y);
    }
    __syncthreads();
    for (u32 s = 0; s < logN; ++s) {
        const u32 lh = logN - 1 - s, half = 1u << lh;
        for (u32 b = threadIdx.x; b < n; b += FFT_THREADS) {
            const u32 j = b & (half - 1), i0 = ((b >> lh) << (lh + 1)) + j, i1 = i0 + half;
            const double2 x = tile[i0], y = tile[i1];
            tile[i0] = cadd(x, y);
            tile[i1] = cmul(csub(x, y), tw[half + j]);
        }
        __syncthreads();
    }
    for (u32 k = threadIdx.x; k < (real ? n : N); k += FFT_THREADS) coef.put(k, tile[__brev(k) >> (32 - logN)]);
}

static int fft_tables(ckks_params *P) {
    if (P->d_fft) return CKKS_OK;
    const u32 N = P->N, n = N / 2;
    const size_t words = 2 * ((size_t)n + N + N) + (n + 256) / 2;           // see ckks_params::d_fft
    std::vector<double> tab(words, 0.0);
    double *dec = tab.data(), *enc = dec + 2 * (size_t)n, *twist = enc + 2 * (size_t)N;
    u32 *bin = reinterpret_cast<u32 *>(twist + 2 * (size_t)N), *colmap = bin + n;
    const long double pi = 3.14159265358979323846264338327950288L;
    for (u32 h = 1; h < n; h *= 2) {
        u32 e = 1;                                          // 5^j mod 8h
        for (u32 j = 0; j < h; ++j) {
            const long double a = 2 * pi * e / (8.0L * h);
            dec[2 * (h + j)] = (double)cosl(a);
            dec[2 * (h + j) + 1] = (double)sinl(a);
            e = e * 5 % (8 * h);
        }
    }
    // the N-th roots of the last half length, every 2^s-th of them for the shorter ones
    for (u32 e = 0; e < n; ++e) {
        enc[2 * (n + e)] = (double)cosl(2 * pi * e / N);
        enc[2 * (n + e) + 1] = (double)-sinl(2 * pi * e / N);
    }
    for (u32 h = n / 2; h >= 1; h /= 2)
        for (u32 j = 0; j < h; ++j) {
            enc[2 * (h + j)] = enc[2 * (n + j * (n / h))];
            enc[2 * (h + j) + 1] = enc[2 * (n + j * (n / h)) + 1];
        }
    for (u32 k = 0; k < N; ++k) {
        twist[2 * k] = (double)cosl(pi * k / N);
        twist[2 * k + 1] = (double)-sinl(pi * k / N);
    }
    u64 e = 1;
    for (u32 j = 0; j < n; ++j) {
        bin[j] = (u32)((e - 1) >> 1);
        e = e * 5 % (2ull * N);
    }
    if (P->logN > 12) {
        const u32 cols = FFT_TILE >> (P->logN - 8), sc = cols / 2;          // columns of a far group
        for (u32 pl = 0; pl < 256; ++pl) {
            const u32 x = pl % cols, t0 = bin[pl / cols * sc + x % sc] & 255;
            colmap[pl] = x < sc ? t0 : 255 - t0;
        }
        std::vector<double> row(512);
        for (u32 b = 1; b < N / 256; ++b) {
            double *w = enc + 512 * (size_t)b;
            std::copy(w, w + 512, row.begin());
            for (u32 pl = 0; pl < 256; ++pl) std::copy_n(row.begin() + 2 * colmap[pl], 2, w + 2 * pl);
        }
    }
    double *d = nullptr;
    CKKS_HIP(hipMalloc(&d, words * sizeof(double)));
    const hipError_t err = hipMemcpy(d, tab.data(), words * sizeof(double), hipMemcpyHostToDevice);
    if (err != hipSuccess) {
        hipFree(d);
        return hip_fail(err, "hipMemcpy (transform tables)");
    }
    P->d_fft = d;
    return CKKS_OK;
}

struct FftTables {
    const double2 *dec, *enc, *twist;
    const u32 *bin, *colmap;
    explicit FftTables(const ckks_params *P)
        : dec((const double2 *)P->d_fft), enc(dec + P->N / 2), twist(enc + P->N), bin((const u32 *)(twist + P->N)),
          colmap(bin + P->N / 2) {}
};

static u64 inv_mod_host(u64 a, u64 q) {   // q prime
    unsigned __int128 r = 1, b = a % q;
    for (u64 e = q - 2; e; e >>= 1) {
        if (e & 1) r = r * b % q;
        b = b * b % q;
    }
    return (u64)r;
}

// The vectors go chunk by chunk, each chunk read whole before any of it is written: in [count][win] words, out
// [count][wout].  What may then happen to buffers that overlap.
enum Overlap { APART, SERVED, REFUSED };   // REFUSED: a chunk would write over words that a later one reads
static Overlap overlap_of(const void *in, size_t win, const void *out, size_t wout, u32 count) {
    if (!words_overlap(in, count * win, out, count * wout)) return APART;
    for (size_t done = ENC_CHUNK; done < count; done += ENC_CHUNK)
        if (words_overlap((const u64 *)in + done * win, (count - done) * win, out, done * wout)) return REFUSED;
    return SERVED;
}

}  // namespace ckks

using namespace ckks;

extern "C" {

int ckks_encode(ckks_params_t *P, const double *d_slots, uint32_t count, double scale, uint32_t flags,
                int64_t *d_coeffs, void *stream_) {
    if (!P || (count && (!d_slots || !d_coeffs))) {
        set_error("ckks_encode: null argument");
        return CKKS_E_INVAL;
    }
    if (!(scale > 0.0) || !std::isfinite(scale) || (flags & ~(uint32_t)CKKS_ENCODE_REAL)) {
        set_error("ckks_encode: scale %g must be positive and finite, flags 0x%x must be known", scale, flags);
        return CKKS_E_INVAL;
    }
    if (count == 0) return CKKS_OK;
    const Overlap lap = overlap_of(d_slots, P->N, d_coeffs, P->N, count);
    if (lap == REFUSED) {
        set_error("ckks_encode: d_coeffs overlaps slots that are read after it is written");
        return CKKS_E_INVAL;
    }
    hipStream_t stream = (hipStream_t)stream_;
    int rc = fft_tables(P);
    if (rc) return rc;
    const u32 N = P->N, n = N / 2, chunk = std::min<u32>(count, ENC_CHUNK);
    const u32 real = flags & CKKS_ENCODE_REAL;
    const bool aside = lap != APART && P->logN <= 12;     // one kernel reads and writes: its results wait in the scratch
    const FftTables ft(P);
    rc = P->ensure_scratch((size_t)chunk * N * sizeof(double2), stream);
    if (rc) return rc;
    double2 *v = (double2 *)P->d_scratch;
    for (u32 done = 0; done < count; done += chunk) {
        const u32 c = std::min(chunk, count - done);
        const double2 *slots = (const double2 *)d_slots + (size_t)done * n;
        int64_t *coeffs = d_coeffs + (size_t)done * N;
        const EncodeOut out{aside ? (int64_t *)v : coeffs, ft.twist, N, real, scale / N};
#define FAR_LAUNCH(S)                                                                                                \
    hipLaunchKernelGGL(encode_far_kernel<S>, dim3(1u << (S - 4), c), dim3(ENC_THREADS), 0, stream, slots, v, ft.enc, \
                       ft.bin, real)
        switch (P->logN) {
            case 13: FAR_LAUNCH(5); break;
            case 14: FAR_LAUNCH(6); break;
            case 15: FAR_LAUNCH(7); break;
            case 16: FAR_LAUNCH(8); break;
            case 17: FAR_LAUNCH(9); break;
            default:
                hipLaunchKernelGGL(encode_small_kernel, dim3(c), dim3(FFT_THREADS), 0, stream, slots, ft.enc, ft.bin, out,
                                   P->logN, real);
        }
#undef FAR_LAUNCH
        CKKS_LAUNCH_CHECK("encode_far_kernel");
        if (aside) CKKS_HIP(hipMemcpyAsync(coeffs, v, (size_t)c * N * sizeof(u64), hipMemcpyDeviceToDevice, stream));
        if (P->logN > 12) {
            hipLaunchKernelGGL(encode_near_kernel, dim3(N / FFT_TILE, c), dim3(ENC_THREADS), 0, stream, v, ft.enc,
                               ft.colmap, out, P->logN);
            CKKS_LAUNCH_CHECK("encode_near_kernel");
        }
    }
    return CKKS_OK;
}

int ckks_decode(ckks_params_t *P, const uint64_t *d_res, uint32_t nlimbs, uint32_t count, double scale,
                double *d_slots, void *stream_) {
    if (!P || (count && (!d_res || !d_slots))) {
        set_error("ckks_decode: null argument");
        return CKKS_E_INVAL;
    }
    if (nlimbs < 1 || nlimbs > 2 || nlimbs > P->L) {
        set_error("ckks_decode: nlimbs = %u, must be 1 or 2 and at most L = %u", nlimbs, P->L);
        return CKKS_E_INVAL;
    }
    if (!(scale > 0.0) || !std::isfinite(scale)) {
        set_error("ckks_decode: scale %g must be positive and finite", scale);
        return CKKS_E_INVAL;
    }
    if (count == 0) return CKKS_OK;
    const Overlap lap = overlap_of(d_res, (size_t)nlimbs * P->N, d_slots, P->N, count);
    if (lap == REFUSED) {
        set_error("ckks_decode: d_slots overlaps residues that are read after it is written");
        return CKKS_E_INVAL;
    }
    const bool aside = lap != APART && P->logN <= 12;     // as in ckks_encode
    hipStream_t stream = (hipStream_t)stream_;
    int rc = fft_tables(P);
    if (rc) return rc;
    const u32 N = P->N, n = N / 2, logn = P->logN - 1, chunk = std::min<u32>(count, ENC_CHUNK);
    const FftTables ft(P);
    rc = P->ensure_scratch((size_t)chunk * n * sizeof(double2), stream);
    if (rc) return rc;
    double2 *v = (double2 *)P->d_scratch;
    const u64 q0 = P->mod[0], q1 = nlimbs > 1 ? P->mod[1] : 0;
    ModConst m1 = nlimbs > 1 ? P->hmod[1] : P->hmod[0];
    u64 q0inv = 0;
    double q0inv_fp = 0.0;
    if (nlimbs > 1) {
        const unsigned __int128 inv = inv_mod_host(q0 % q1, q1);
        q0inv = (u64)((inv << 64) % q1);                 // Montgomery form: times 2^64 mod q1
        if (((q0 | q1) >> 50) == 0) q0inv_fp = (double)(u64)inv;
    }
    const size_t stride = (size_t)nlimbs * N;
    for (u32 done = 0; done < count; done += chunk) {
        const u32 c = std::min(chunk, count - done);
        double2 *slots = (double2 *)d_slots + (size_t)done * n;
        const DecodeIn in{d_res + done * stride, n, nlimbs, q0, q1, q0inv, m1, q0inv_fp, nlimbs > 1 ? 1.0 / (double)q1 : 0.0};
        const bool deal = c >= 8 && P->logN >= 14 && P->logN <= 16;      // see deal_vectors
#define FAR_LAUNCH(S)                                                                                                \
    hipLaunchKernelGGL((deal ? decode_far_kernel<S, true> : decode_far_kernel<S, false>), dim3(1u << (S - 4), c),     \
                       dim3(FFT_THREADS), 0, stream, v, slots, ft.dec, 1.0 / scale)
        if (n >= FFT_TILE) {
            // a workgroup of either kind per CU or less: 5 / 16 / 32 / 64 vectors at 2^15 (20 to 256 workgroups) 14.5 / 15.9 /
            // 20.3 / 24.5 us by 256 threads, 13.6 / 14.5 / 18.1 / 22.6 by 1024; 48 at 2^16 (384) 28.8 and 29.8
            const bool wide = n / FFT_TILE * c <= 256;
            hipLaunchKernelGGL(wide ? (deal ? decode_near_wide_kernel<true> : decode_near_wide_kernel<false>)
                               : (deal ? decode_near_kernel<true> : decode_near_kernel<false>),
                               dim3(n / FFT_TILE, c),
                               dim3(wide ? 1024 : FFT_THREADS), 0, stream, v, ft.dec, in, stride, logn);
            CKKS_LAUNCH_CHECK("decode_near_kernel");
        }
        switch (P->logN) {
            case 13: FAR_LAUNCH(4); break;
            case 14: FAR_LAUNCH(5); break;
            case 15: FAR_LAUNCH(6); break;
            case 16: FAR_LAUNCH(7); break;
            case 17: FAR_LAUNCH(8); break;
            default:
                hipLaunchKernelGGL(decode_small_kernel, dim3(c), dim3(FFT_THREADS), 0, stream, aside ? v : slots, ft.dec, in,
                                   stride, logn, 1.0 / scale);
        }
#undef FAR_LAUNCH
        CKKS_LAUNCH_CHECK("decode_far_kernel");
        if (aside) CKKS_HIP(hipMemcpyAsync(slots, v, (size_t)c * n * sizeof(double2), hipMemcpyDeviceToDevice, stream));
    }
    return CKKS_OK;
}

}  // extern "C"
