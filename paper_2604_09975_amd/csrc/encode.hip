// Complex-slot encode / decode on the device (Sec. 2.1 Encode / Decode, Sec. 3.1 slot order).
// Slot j of a plaintext m(X) is m(zeta^(5^j)), zeta = exp(i*pi/N), j < n = N/2.  With w_k = m_k + i*m_(k+n), k < n,
// zeta^(5^j n) = i gives z_j = sum_k w_k zeta^(5^j k): n complex values in, n out.  Since 5^(n/2) = 1 + N (mod 2N), the
// sum splits into the even and the odd k like an FFT,
//   z_j, z_(j+n/2) = E_j +- zeta^(5^j) O_j,   j < n/2,
// with E, O the same transform at half the length (5^j modulo a quarter of the roots each time).  Decode runs these
// butterflies from length 2 up to n, on w in bit-reversed order; encode runs their inverses from n down to 2.  The slots
// are in order on their side without a permutation, and the twiddle of butterfly j of half length h is
// tw[h + j] = exp(2*pi*i*(5^j mod 8h)/(8h)).
//
// n >= 4096: two passes over 4096-element tiles, 16 elements per thread, at most four stages (radix 16) between exchanges
// through LDS:
//   far:  the stages of half length 256 and more, on columns (elements 256 apart), 2^S = n/256 rows of 4096 >> S columns;
//         slots on one side, the scratch array on the other.
//   near: the stages of half length up to 128, on 16 runs of 256 elements that lie n/16 apart: then the tile's k = bitrev(p)
//         form runs of 16, a 128-byte line of the coefficients that are on the other side.
// A pass reads and writes every element once, and nothing else touches memory.  n < 4096: one workgroup per vector.
// Off the server's hot path.  96 real vectors at N = 2^16: 308 us with an N-point FFT between separate permutation, twist
// and rounding kernels, 46 us now (4 TB/s over what it moves); 5 vectors decoded at N = 2^15: 45 us, 14 us now.
#include <cmath>

#include "ckks_internal.h"
#include "common_kernels.h"
#include "mac_device.h"

namespace ckks {

constexpr u32 FFT_THREADS = 256;
constexpr u32 FFT_TILE = 4096;
constexpr u32 ENC_CHUNK = 128;        // vectors transformed per scratch chunk (N = 2^16: 64 MiB)
// tile element i: one pad element after 16 and one after 256, so that runs of 16, strides of 16 and strides of 256 all
// fall on distinct banks.  70 KB: two workgroups per CU.
__device__ __forceinline__ u32 fft_slot(u32 i) { return i + (i >> 4) + (i >> 8); }
constexpr u32 FFT_LDS = FFT_TILE + FFT_TILE / 16 + FFT_TILE / 256;

__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
    return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ double2 cmul_conj(double2 a, double2 b) {     // a * conj(b)
    return make_double2(a.x * b.x + a.y * b.y, a.y * b.x - a.x * b.y);
}
__device__ __forceinline__ double2 cadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ double2 csub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }

// LOGR stages on elements off + r * stride, r < 2^LOGR, of every block of 2^LOGR * stride: half lengths
// stride << (LOGR-1) .. stride (INV: encode) or the other way round (decode)
template <u32 LOGR, bool INV>
__device__ __forceinline__ void fft_group(double2 *v, const double2 *__restrict__ tw, u32 stride, u32 off) {
    constexpr u32 R = 1u << LOGR;
#pragma unroll
    for (u32 s = 0; s < LOGR; ++s) {
        const u32 t = INV ? s : LOGR - 1 - s, g = R >> (t + 1);
#pragma unroll
        for (u32 i = 0; i < g; ++i) {
            const double2 w = tw[(g + i) * stride + off];
#pragma unroll
            for (u32 k = 0; k < (1u << t); ++k) {
                double2 &a = v[k * 2 * g + i], &b = v[k * 2 * g + i + g];
                const double2 x = a, y = INV ? b : cmul(b, w);
                a = cadd(x, y);
                b = INV ? cmul_conj(csub(x, y), w) : csub(x, y);
            }
        }
    }
}

// Where the coefficients meet the transform: w_k out of / into the caller's array.
struct EncodeOut {
    int64_t *c;                // the vector's N coefficients
    u32 n, real;
    double mul;
    // Nearest integers to scale * m.  A real slot vector is fixed by conjugation, so its polynomial satisfies
    // m[N-k] = -m[k] and m[N/2] = 0 exactly; real != 0 imposes that on the rounded values (the transform gives it only
    // up to rounding).
    __device__ __forceinline__ void put(u32 k, double2 w) const {
        const int64_t re = (int64_t)rint(w.x * mul);
        c[k] = re;
        if (real)
            c[k ? 2 * n - k : n] = k ? -re : 0;
        else
            c[n + k] = (int64_t)rint(w.y * mul);
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

// far pass (see the head of the file).  INV: slots -> scratch; else scratch -> slots, times inv_scale.
// grid: x = group of 4096 >> S columns, y = vector
template <u32 S, bool INV>
__global__ __launch_bounds__(FFT_THREADS) void fft_far_kernel(const double2 *__restrict__ in, double2 *__restrict__ out,
                                                              const double2 *__restrict__ tw, u32 real,
                                                              double inv_scale) {
    constexpr u32 COLS = FFT_TILE >> S, LOW = S - 4, SUB = 1u << LOW, n = 256u << S;
    __shared__ double2 tile[FFT_LDS];
    const u32 col = threadIdx.x % COLS, q = threadIdx.x / COLS;              // q < SUB
    const u32 pcol = blockIdx.x * COLS + col;
    const double2 *src = in + (size_t)blockIdx.y * n + pcol;
    double2 *dst = out + (size_t)blockIdx.y * n + pcol;
    double2 v[16];
    // rows r * SUB + q: the top four row bits; rows (q + SUB * m) * SUB + r, r < SUB: the others
    auto top_row = [&](u32 r) { return r * SUB + q; };
    auto low_row = [&](u32 e) { return (q + SUB * (e >> LOW)) * SUB + (e & (SUB - 1)); };
    auto top = [&]() { fft_group<4, INV>(v, tw, SUB * 256, q * 256 + pcol); };
    auto low = [&]() {
        if constexpr (LOW > 0) {
#pragma unroll
            for (u32 m = 0; m < (16u >> LOW); ++m) fft_group<LOW, INV>(v + m * SUB, tw, 256, pcol);
        }
    };
    if (INV) {
#pragma unroll
        for (u32 r = 0; r < 16; ++r) {
            v[r] = src[top_row(r) * 256];
            if (real) v[r].y = 0.0;
        }
        top();
        if constexpr (LOW > 0) {
#pragma unroll
            for (u32 r = 0; r < 16; ++r) tile[fft_slot(top_row(r) * COLS + col)] = v[r];
            __syncthreads();
#pragma unroll
            for (u32 e = 0; e < 16; ++e) v[e] = tile[fft_slot(low_row(e) * COLS + col)];
            low();
        }
#pragma unroll
        for (u32 e = 0; e < 16; ++e) dst[low_row(e) * 256] = v[e];
    } else {
#pragma unroll
        for (u32 e = 0; e < 16; ++e) v[e] = src[low_row(e) * 256];
        if constexpr (LOW > 0) {
            low();
#pragma unroll
            for (u32 e = 0; e < 16; ++e) tile[fft_slot(low_row(e) * COLS + col)] = v[e];
            __syncthreads();
#pragma unroll
            for (u32 r = 0; r < 16; ++r) v[r] = tile[fft_slot(top_row(r) * COLS + col)];
        }
        top();
#pragma unroll
        for (u32 r = 0; r < 16; ++r) dst[top_row(r) * 256] = make_double2(v[r].x * inv_scale, v[r].y * inv_scale);
    }
}

// near pass: INV: scratch -> coefficients (EncodeOut); else residues (DecodeIn) -> scratch.
// grid: x = n / 4096, y = vector
template <bool INV, class Coef>
__global__ __launch_bounds__(FFT_THREADS) void fft_near_kernel(double2 *__restrict__ scratch,
                                                               const double2 *__restrict__ tw, Coef first,
                                                               size_t coef_stride, u32 logn) {
    __shared__ double2 tile[FFT_LDS];
    const u32 tid = threadIdx.x, h = tid >> 4, c = tid & 15, f = blockIdx.x, fb = logn - 12;
    double2 *v0 = scratch + ((size_t)blockIdx.y << logn) + (((h << fb) + f) << 8);     // run h of the tile
    Coef coef = first;
    if constexpr (INV)
        coef.c += blockIdx.y * coef_stride;
    else
        coef.r += blockIdx.y * coef_stride;
    // coefficient side: thread (m & 15 = h, hh = c) holds element lo = bitrev8(m) of run bitrev4(hh), k as below
    const u32 ch = __brev(c) >> 28, fk = (fb ? __brev(f) >> (32 - fb) : 0) * 16 + c;
    auto side = [&](u32 r) { return fft_slot(ch * 256 + (__brev(h + 16 * r) >> 24)); };
    auto kidx = [&](u32 r) { return ((h + 16 * r) << (logn - 8)) + fk; };
    double2 v[16];
    if constexpr (INV) {
#pragma unroll
        for (u32 r = 0; r < 16; ++r) v[r] = v0[c + 16 * r];
        fft_group<4, true>(v, tw, 16, c);
#pragma unroll
        for (u32 r = 0; r < 16; ++r) tile[fft_slot(h * 256 + c + 16 * r)] = v[r];
        __syncthreads();
#pragma unroll
        for (u32 r = 0; r < 16; ++r) v[r] = tile[fft_slot(h * 256 + c * 16 + r)];
        fft_group<4, true>(v, tw, 1, 0);
#pragma unroll
        for (u32 r = 0; r < 16; ++r) tile[fft_slot(h * 256 + c * 16 + r)] = v[r];      // a thread's own slots
        __syncthreads();
#pragma unroll
        for (u32 r = 0; r < 16; ++r) coef.put(kidx(r), tile[side(r)]);
    } else {
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
        for (u32 r = 0; r < 16; ++r) tile[fft_slot(h * 256 + c * 16 + r)] = v[r];      // a thread's own slots
        __syncthreads();
#pragma unroll
        for (u32 r = 0; r < 16; ++r) v[r] = tile[fft_slot(h * 256 + c + 16 * r)];
        fft_group<4, false>(v, tw, 16, c);
#pragma unroll
        for (u32 r = 0; r < 16; ++r) v0[c + 16 * r] = v[r];
    }
}

// n < 4096: the whole transform of one vector in LDS, one exchange per stage.  grid: x = vector
template <bool INV, class Coef>
__global__ __launch_bounds__(FFT_THREADS) void fft_small_kernel(const double2 *__restrict__ in, double2 *__restrict__ out,
                                                                const double2 *__restrict__ tw, Coef first,
                                                                size_t coef_stride, u32 logn, u32 real,
                                                                double inv_scale) {
    __shared__ double2 tile[FFT_TILE / 2];
    const u32 n = 1u << logn;
    Coef coef = first;
    if constexpr (INV)
        coef.c += blockIdx.x * coef_stride;
    else
        coef.r += blockIdx.x * coef_stride;
    for (u32 i = threadIdx.x; i < n; i += FFT_THREADS) {
        double2 v;
        if constexpr (INV) {
            v = in[(size_t)blockIdx.x * n + i];
            if (real) v.y = 0.0;
        } else {
            v = coef.get(coef.load(__brev(i) >> (32 - logn)));
        }
        tile[i] = v;
    }
    __syncthreads();
    for (u32 s = 0; s < logn; ++s) {
        const u32 lh = INV ? logn - 1 - s : s, half = 1u << lh;
        for (u32 b = threadIdx.x; b < n / 2; b += FFT_THREADS) {
            const u32 j = b & (half - 1), i0 = ((b >> lh) << (lh + 1)) + j, i1 = i0 + half;
            const double2 w = tw[half + j], x = tile[i0], y = INV ? tile[i1] : cmul(tile[i1], w);
            tile[i0] = cadd(x, y);
            tile[i1] = INV ? cmul_conj(csub(x, y), w) : csub(x, y);
        }
        __syncthreads();
    }
    for (u32 i = threadIdx.x; i < n; i += FFT_THREADS) {
        const double2 v = tile[i];
        if constexpr (INV)
            coef.put(__brev(i) >> (32 - logn), v);
        else
            out[(size_t)blockIdx.x * n + i] = make_double2(v.x * inv_scale, v.y * inv_scale);
    }
}

static int fft_tables(ckks_params *P) {
    if (P->d_fft_tw) return CKKS_OK;
    const u32 n = P->N / 2;
    std::vector<double> w(2 * (size_t)n, 0.0);
    const long double pi = 3.14159265358979323846264338327950288L;
    for (u32 h = 1; h < n; h *= 2) {
        u32 e = 1;                                          // 5^j mod 8h
        for (u32 j = 0; j < h; ++j) {
            const long double a = 2 * pi * e / (8.0L * h);
            w[2 * (h + j)] = (double)cosl(a);
            w[2 * (h + j) + 1] = (double)sinl(a);
            e = e * 5 % (8 * h);
        }
    }
    double *d_w = nullptr;
    CKKS_HIP(hipMalloc(&d_w, w.size() * sizeof(double)));
    hipError_t e_w = hipMemcpy(d_w, w.data(), w.size() * sizeof(double), hipMemcpyHostToDevice);
    if (e_w != hipSuccess) {
        hipFree(d_w);
        return hip_fail(e_w, "hipMemcpy (transform roots)");
    }
    P->d_fft_tw = d_w;
    return CKKS_OK;
}

// the far pass of a ring of 2^13 and more
template <bool INV>
static void launch_far(const ckks_params *P, const double2 *in, double2 *out, u32 count, u32 real, double inv_scale,
                       hipStream_t stream) {
    const double2 *tw = (const double2 *)P->d_fft_tw;
#define FAR_LAUNCH(S)                                                                                              \
    hipLaunchKernelGGL((fft_far_kernel<S, INV>), dim3(1u << (S - 4), count), dim3(FFT_THREADS), 0, stream, in, out, \
                       tw, real, inv_scale)
    switch (P->logN) {
        case 13: FAR_LAUNCH(4); break;
        case 14: FAR_LAUNCH(5); break;
        case 15: FAR_LAUNCH(6); break;
        case 16: FAR_LAUNCH(7); break;
        case 17: FAR_LAUNCH(8); break;
    }
#undef FAR_LAUNCH
}

static u64 inv_mod_host(u64 a, u64 q) {   // q prime
    unsigned __int128 r = 1, b = a % q;
    for (u64 e = q - 2; e; e >>= 1) {
        if (e & 1) r = r * b % q;
        b = b * b % q;
    }
    return (u64)r;
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
    hipStream_t stream = (hipStream_t)stream_;
    int rc = fft_tables(P);
    if (rc) return rc;
    const u32 N = P->N, n = N / 2, logn = P->logN - 1, chunk = std::min<u32>(count, ENC_CHUNK);
    const u32 real = flags & CKKS_ENCODE_REAL;
    const double2 *tw = (const double2 *)P->d_fft_tw;
    rc = P->ensure_scratch((size_t)chunk * n * sizeof(double2), stream);
    if (rc) return rc;
    double2 *v = (double2 *)P->d_scratch;
    for (u32 done = 0; done < count; done += chunk) {
        const u32 c = std::min(chunk, count - done);
        const double2 *slots = (const double2 *)d_slots + (size_t)done * n;
        const EncodeOut out{d_coeffs + (size_t)done * N, n, real, scale / n};
        if (n >= FFT_TILE) {
            launch_far<true>(P, slots, v, c, real, 1.0, stream);
            CKKS_LAUNCH_CHECK("fft_far_kernel");
            hipLaunchKernelGGL((fft_near_kernel<true, EncodeOut>), dim3(n / FFT_TILE, c), dim3(FFT_THREADS), 0, stream, v,
                               tw, out, (size_t)N, logn);
            CKKS_LAUNCH_CHECK("fft_near_kernel");
        } else {
            hipLaunchKernelGGL((fft_small_kernel<true, EncodeOut>), dim3(c), dim3(FFT_THREADS), 0, stream, slots, nullptr,
                               tw, out, (size_t)N, logn, real, 1.0);
            CKKS_LAUNCH_CHECK("fft_small_kernel");
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
    hipStream_t stream = (hipStream_t)stream_;
    int rc = fft_tables(P);
    if (rc) return rc;
    const u32 N = P->N, n = N / 2, logn = P->logN - 1, chunk = std::min<u32>(count, ENC_CHUNK);
    const double2 *tw = (const double2 *)P->d_fft_tw;
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
        if (n >= FFT_TILE) {
            hipLaunchKernelGGL((fft_near_kernel<false, DecodeIn>), dim3(n / FFT_TILE, c), dim3(FFT_THREADS), 0, stream, v,
                               tw, in, stride, logn);
            CKKS_LAUNCH_CHECK("fft_near_kernel");
            launch_far<false>(P, v, slots, c, 0, 1.0 / scale, stream);
            CKKS_LAUNCH_CHECK("fft_far_kernel");
        } else {
            hipLaunchKernelGGL((fft_small_kernel<false, DecodeIn>), dim3(c), dim3(FFT_THREADS), 0, stream, nullptr, slots,
                               tw, in, stride, logn, 0u, 1.0 / scale);
            CKKS_LAUNCH_CHECK("fft_small_kernel");
        }
    }
    return CKKS_OK;
}

}  // extern "C"
