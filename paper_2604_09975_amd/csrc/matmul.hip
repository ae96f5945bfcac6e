// The projection kernel Y = XW on ciphertexts (Sec. 3.2, App. A.2) and rescale (Sec. 2.2).
//
//   bank     x_q^(g) = rot(x^(g); q*m), q < N1            one hoisted call per input group
//   diagonal acc_{b,p} = sum_g sum_q x_q^(g) (.) w_{b,p,g,q}  the byte mover: every weight limb is read once
//   giant    y_b = acc_{b,0} + sum_{p>=1} rot(acc_{b,p}; p*N1*m)
//   bias     y_b.c0 += bias_b
// Real packing: the imaginary half of the complex weights of App. A.2.1 is not used.
#include <algorithm>

#include "ckks_internal.h"
#include "common_kernels.h"
#include "mac_device.h"
#include "ntt_device.h"

namespace ckks {

constexpr u32 MM_THREADS = 256;
constexpr u32 MM_TB = 8;   // (b,p) accumulators kept in registers per thread on primes of 50 bits and more

// int64 coefficients [count][N] -> canonical residues [count][level][N]
__global__ __launch_bounds__(EW_THREADS) void expand_coeffs_kernel(const int64_t *__restrict__ coef,
                                                                   u64 *__restrict__ out,
                                                                   const ModConst *__restrict__ mods, u32 level,
                                                                   u32 N) {
    const u32 n = blockIdx.x * EW_THREADS + threadIdx.x;
    const u32 d = blockIdx.y;
    const int64_t v = coef[(size_t)d * N + n];
    for (u32 i = 0; i < level; ++i) out[((size_t)d * level + i) * N + n] = reduce_signed(v, mods[i]);
}

// The same with the first pass of the forward transform (rings of 2^12 and more): row (d, i) of out leaves as the column
// pass (LOGR stages) or, at N = 2^12 (LOGR = 0), the whole transform of coefficient vector d modulo limb i would leave it.
// The canonical residues never reach memory: 32 vectors on 9 limbs at 2^15 took 16 + 18 us for the two kernels this
// replaces, 26 us for this one (the call 71 and 55 us).
// grid: x = workgroups of a column pass (tiles), y = d * level + i: the limbs of a vector follow each other and find its
// coefficients in L2.
template <u32 LOGR>
__global__ __launch_bounds__(NTT_THREADS) void expand_pass_kernel(const int64_t *__restrict__ coef, u64 *__restrict__ out,
                                                                  const ModConst *__restrict__ mods,
                                                                  const ModFp *__restrict__ modf,
                                                                  const u64 *__restrict__ tws,
                                                                  const double *__restrict__ twf,
                                                                  const u64 *__restrict__ ninvs, u32 level) {
    constexpr u32 logN = 12 + LOGR;
    __shared__ u64 lds[LOGR ? 1 : Tile<4>::WORDS];
    const u32 d = uniform_div(blockIdx.y, level), i = blockIdx.y - d * level;
    const ModConst m = mods[i];
    const ModFp mf = modf[i];
    const int64_t *src = coef + ((size_t)d << logN);
    u64 *dst = out + ((size_t)blockIdx.y << logN);
    auto load = [&](u32 idx) { return reduce_signed(src[idx], m); };
    auto store = [&](u32 idx, u64 v) { dst[idx] = v; };
    auto load_a = [&](u32 at, u32 col) { return reduce_signed((src + at)[col], m); };
    auto store_a = [&](u32 at, u32 col, u64 v) { (dst + at)[col] = v; };
    auto go = [&](const auto &f) {
        if constexpr (LOGR == 0) {
            pass_b_body<false>(f, logN, lds, load, store);
        } else {
            constexpr u32 COLS = LOGR < 4 ? 16u >> LOGR : 1;
#pragma unroll
            for (u32 c = 0; c < COLS; ++c)
                pass_a_body<false, LOGR>(f, (c * gridDim.x + blockIdx.x) * NTT_THREADS + threadIdx.x, load_a, store_a);
        }
    };
    with_field(mf, mods, tws, twf, ninvs, i, logN, go);
}

// rows [rows][N], row r modulo limb r % level: x <- x * c mod q (c canonical, any size)
__global__ __launch_bounds__(EW_THREADS) void scale_rows_kernel(u64 *data, const ModConst *__restrict__ mods,
                                                                u32 level, u32 N, u64 c) {
    const u32 n = blockIdx.x * EW_THREADS + threadIdx.x;
    const u32 row = blockIdx.y;
    const ModConst m = mods[row % level];
    const u64 cm = mont_mul(reduce_any(c, m), m.r2, m);
    const size_t idx = (size_t)row * N + n;
    data[idx] = mont_mul(data[idx], cm, m);
}

// ---- acc[bp][comp][i][k] = sum_{gq} bank[gq][comp][i][k] * w[bp][gq][i][k] ------------------------------------------
//
// Operands.  On primes below 2^50 bank residues and weights are balanced, |x|, |w| <= (q+1)/2 <= 2^49, exact in doubles:
// the key switches store the bank that way (SwitchItem::balanced), the unpacked weight store holds the doubles, and a
// packed record holds w + 2^49.  Larger primes keep canonical bank residues and Montgomery weights (diag_mac_int_kernel).
//
// Packed weight records: 50 bits per residue, in the order in which a wavefront reads them, so that it has one stream:
// [limb][chunk of 128 residues][tile of TB pairs][gq / 4][pair of the tile][3200 bytes].  A 3200-byte record holds the
// chunk's residues of four steps: two parts of 16 bytes per lane (residues 2l, 2l+1 of two steps, low 32 bits), two of 8
// bytes per lane (bits 32..47) and one of 4 bytes per pair of lanes (bits 48, 49; one byte per step), each a whole
// number of 128-byte lines read by one load of the wavefront.  The steps behind the last whole record follow in an area of
// their own, one 800-byte record per step ([limb][chunk][tile][step][pair]: 512 + 256 + 32 bytes), and a last tile of
// fewer pairs holds those alone, so that nothing is stored or read for padding.  A half store holds the first N/2 residues
// of a limb (real diagonals: the rest is the mirror image), a whole store all N.
// What the order is worth, QKV layer (38 GB): parts that share lines 9.6 ms, whole lines with every pair's records in a
// place of their own 8.54 ms, this order 8.43 ms.  What the exact sizes are worth, 24 limbs at 2^16, real diagonals: 64 steps
// of one pair 539 us with tile and record filled up, 374 now; 5 steps of 16 pairs 227 and 188; 7 steps of 9 pairs 174 and 145.
constexpr u32 TB = 4;                                              // (b,p) pairs of a tile
constexpr u32 REC_BYTES = 3200, REC_CHUNK = 128, REC_MID = 2048, REC_TOP = 3072;
constexpr u32 STEP_BYTES = 800, STEP_MID = 512, STEP_TOP = 768;    // the record of a single step
struct PackedShape {
    u32 GQ, BP, nch, level;                                        // steps, pairs, chunks per limb
    __host__ __device__ u32 records() const { return GQ / 4; }     // whole ones, per pair and chunk
    // pairs of the tile of pair bp, and where their r-th records (or the records of step 4 * records() + r) lie
    __host__ __device__ u32 pairs(u32 bp) const { return BP - bp / TB * TB < TB ? BP - bp / TB * TB : TB; }
    __host__ __device__ size_t rec(u32 bp, u32 i, u32 chunk, u32 r) const {
        return ((((size_t)i * nch + chunk) * BP + bp / TB * TB) * records() + (size_t)r * pairs(bp) + bp % TB) * REC_BYTES;
    }
    __host__ __device__ size_t step(u32 bp, u32 i, u32 chunk, u32 r) const {
        return (size_t)level * nch * BP * records() * REC_BYTES +
               ((((size_t)i * nch + chunk) * BP + bp / TB * TB) * (GQ % 4) + (size_t)r * pairs(bp) + bp % TB) * STEP_BYTES;
    }
    __host__ __device__ size_t bytes() const { return (size_t)level * nch * BP * GQ * STEP_BYTES; }
};
static inline PackedShape packed_shape(u32 N, u32 level, u32 GQ, u32 BP, bool whole) {
    return PackedShape{GQ, BP, (whole ? N : N / 2) / REC_CHUNK, level};
}

// grid: x = tile of TB (b,p) pairs, from the one that holds bp0, y = run of 512 coefficients (SYM: and their mirrors), z = limb (limbs.id:
// the limbs this launch covers).  A thread owns two adjacent coefficients k, k+1 and NP pairs, of which those from bp0 to
// bp1 - 1 are read and stored; two steps' weights and two steps' bank residues are on their way while two are multiplied.
// SYM: plaintexts that encode REAL slot vectors.  Such a polynomial is fixed by X -> X^-1, so its transform is a
// palindrome: w[k] = w[N-1-k] (the exponents 2*bitrev(k)+1 and 2*bitrev(N-1-k)+1 are negatives of each other mod 2N).
// Only the first half of every weight limb is read; each value serves coefficient k and its mirror: the thread owns
// N-2-k, N-1-k as well.
// TB = 4: 32 outputs of two doubles (128 registers) are what two waves per SIMD leave room for.
// NP: pairs a thread computes.  A lone tile of one or two pairs takes an instance of that many (109 and 154 registers instead
// of 250, no products for absent pairs) while the bank fits the Infinity Cache and latency counts: 24 limbs at 2^16, one pair
// of 1 / 5 / 8 steps 18.4 / 43 / 52 us with NP = 4, 13.5 / 32 / 48 with NP = 1.  Larger banks are a stream, and more
// wavefronts on it do not help: 16 steps, general diagonals, 128 us with NP = 4, 138 with NP = 1.
// Steps gq0 .. gq1-1 of the GQ per pair are summed; accumulate: onto what acc already holds.
// swizzle: workgroups go to the XCDs round-robin and each XCD has its own L2, so the linear workgroup id is unfolded to
// let one XCD walk all (b,p) tiles of a run of coefficients back to back: the bank lines of that run are then fetched
// into one L2 once.
// SH = 2, 4 (packed stores; share_of): SH wavefronts of a workgroup take consecutive tiles of one chunk of 128 coefficients and
// share its bank residues, two steps at a time, through LDS (16 KiB): each brings 1 / SH of them two steps ahead.  The bank then
// crosses from L2 to the CUs once per SH tiles and is fetched into L2 less often; the records go past L2's replacement order
// (7818 -> 7742 us).  Every wavefront of a workgroup runs every step, those beyond the last tile for the barriers alone.  (Waves
// that read the bank through the vector L1 together, without LDS, take 12 to 19 ms.)
// What bounds it (QKV layer, 34.0 GB of records, 2.4 GB of bank, 1.8 GB of sums): memory, 4.95 TB/s with SH = 4, 7.74 ms; 8.43
// ms with a bank stream for each wavefront (8.32 to 8.47 from card to card), an earlier form of which, 8.45 ms, took 8.40
// without the products, 4.36 without the record loads and 7.05 without the bank loads (5.1 TB/s; a plain read reaches 5.3).
// The kernel with a quotient per product was bound by fp64 issue: 8.66 ms with the vector units 92 % busy; these sums keep
// them 62 % busy.
template <bool SYM, bool PACKED, u32 NP, u32 SH = 0>
__global__ __launch_bounds__(MM_THREADS, 2) void diag_mac_kernel(const double *__restrict__ bank,
                                                              const void *__restrict__ w, u64 *__restrict__ acc,
                                                              const ModFp *__restrict__ modf, LimbIds limbs,
                                                              u32 level, u32 N, u32 GQ, u32 BP, u32 swizzle,
                                                              u32 gq0, u32 gq1, u32 accumulate, u32 bp0, u32 bp1) {
    constexpr u32 CO = SYM ? 4 : 2, HV = CO / 2;                   // coefficients of a thread, pairs of them
    constexpr int NTW = SH ? 2 : 0;                                // non-temporal
    typedef double dvec_t __attribute__((ext_vector_type(2)));
    typedef u64 vec_t __attribute__((ext_vector_type(2)));
    typedef u32 u32x2 __attribute__((ext_vector_type(2)));
    typedef u32 u32x4 __attribute__((ext_vector_type(4)));
    u32 tile = blockIdx.x, run = blockIdx.y;
    if (swizzle) {
        const u32 lin = blockIdx.y * gridDim.x + blockIdx.x;
        const u32 xcd = lin & 7, slot = lin >> 3;
        const u32 d = uniform_div(slot, gridDim.x);
        tile = slot - d * gridDim.x;
        run = d * 8 + xcd;
    }
    const u32 wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (SH) tile = tile * SH + wave % SH;
    const u32 bpt = (bp0 / TB + tile) * TB;                        // the tile's first pair
    const u32 k = SH ? (run * (4 / SH) + wave / SH) * REC_CHUNK + 2 * lane
                     : (run * MM_THREADS + threadIdx.x) * 2;       // SYM: k < N/2
    const u32 kk[2] = {k, N - 2 - k};                              // SYM: the second holds the mirrors of k+1, k
    const u32 i = limbs.id[blockIdx.z];
    const size_t row = (size_t)i * N, w_stride = (size_t)level * N;
    const double q = modf[i].q, u = modf[i].u;
    MacSum a[NP][2][CO];
#pragma unroll
    for (u32 t = 0; t < NP; ++t)
#pragma unroll
        for (u32 c = 0; c < 2; ++c)
#pragma unroll
            for (u32 e = 0; e < CO; ++e) a[t][c][e] = MacSum{MAC_H0, 0.0};
    if (accumulate) {
#pragma unroll
        for (u32 t = 0; t < NP; ++t)
            if (bpt + t >= bp0 && bpt + t < bp1)
#pragma unroll
                for (u32 c = 0; c < 2; ++c)
#pragma unroll
                    for (u32 h = 0; h < HV; ++h) {
                        const vec_t v = *reinterpret_cast<const vec_t *>(acc + ((size_t)(bpt + t) * 2 + c) * w_stride + row + kk[h]);
                        a[t][c][2 * h].l = (double)v[0];
                        a[t][c][2 * h + 1].l = (double)v[1];
                    }
    }
    dvec_t x[SH ? 1 : 2][2][HV];                                   // [step & 1][component]
    constexpr u32 SHC = SH ? 4 / SH : 1, SEGS = 4 * HV, SEG = SHC * HV;   // chunks, segments of one, segments that a wavefront brings
    __shared__ dvec_t xs[SH ? 2 : 1][SH ? SHC * SEGS * 64 : 1];    // [buffer][chunk][step][component][half][lane]
    dvec_t xg[SEG];
    u32 wr[2][NP][6], wt[2][NP];                                   // two steps' weights as loaded, twice; four steps' top bits
    double wp[2][NP][2];                                           // two steps' weights, unpacked store
    // buffer loads: wavefront-uniform addresses stay in scalar registers, the lanes add 32-bit offsets; and a step outside
    // the range reads zeros (a buffer of no records), so that the loop has no branches
    const PackedShape ps{GQ, BP, (SYM ? N / 2 : N) / REC_CHUNK, level};
    const u32 gq_end = PACKED ? min(gq1, 4 * ps.records()) : gq1;  // the steps in whole records; the others come last
    const u32 r_first = gq0 >> 2, r_end = (gq_end + 3) >> 2;       // records of the range
    const double *xp = bank + (size_t)r_first * 8 * w_stride + row;  // the next step to fetch
    auto fetch_x = [&](u32 s, u32 gq) {
        const int bytes = gq >= gq0 && gq < gq_end ? (int)(N * sizeof(double)) : 0;
#pragma unroll
        for (u32 c = 0; c < 2; ++c) {
            const __amdgpu_buffer_rsrc_t rs =
                __builtin_amdgcn_make_buffer_rsrc(const_cast<double *>(xp), 0, bytes, 0x00020000);
#pragma unroll
            for (u32 h = 0; h < HV; ++h)
                x[s][c][h] = __builtin_bit_cast(dvec_t, __builtin_amdgcn_raw_buffer_load_b128(rs, (int)(kk[h] * 8), 0, 0));
            xp += w_stride;
        }
    };
    const u32 top_shift = (lane & 1) * 4;
    const bool live = bpt < bp1;
    // SH: segment wave * SEG + z of two steps' bank residues.  A step outside the range must read zeros here too: the records are
    // of four steps whatever the range, so these residues alone keep its weights out of the sum.  The descriptor is the
    // chunk's own, with no scalar offset, which need not take part in the range check
    auto fetch_shared = [&](u32 g2) {
#pragma unroll
        for (u32 z = 0; z < SEG; ++z) {
            const u32 sg = wave * SEG + z, cw = sg / SEGS, st = sg / (2 * HV) % 2, c = sg / HV % 2, h = sg % HV, gq = 2 * g2 + st;
            const u32 cb = (run * SHC + cw) * REC_CHUNK;
            const int bytes = gq >= gq0 && gq < gq_end ? (int)(REC_CHUNK * sizeof(double)) : 0;
            const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
                const_cast<double *>(bank + ((size_t)gq * 2 + c) * w_stride + row + (h ? N - REC_CHUNK - cb : cb)), 0, bytes, 0x00020000);
            xg[z] = __builtin_bit_cast(dvec_t, __builtin_amdgcn_raw_buffer_load_b128(rs, (int)(lane * 16), 0, 0));
        }
    };
    auto keep_shared = [&](u32 buf) {
#pragma unroll
        for (u32 z = 0; z < SEG; ++z) xs[buf][(wave * SEG + z) * 64 + lane] = xg[z];
    };
    auto take_shared = [&](u32 buf, u32 st) {
#pragma unroll
        for (u32 c = 0; c < 2; ++c)
#pragma unroll
            for (u32 h = 0; h < HV; ++h)
                x[0][c][h] = xs[buf][((wave / (SH ? SH : 1)) * SEGS + (st * 2 + c) * HV + h) * 64 + (h ? 63 - lane : lane)];
    };
    const u32 chunk = __builtin_amdgcn_readfirstlane(k / REC_CHUNK), wpairs = ps.pairs(bpt);
    const unsigned char *wrec = reinterpret_cast<const unsigned char *>(w) + ps.rec(bpt, i, chunk, r_first);
    // pairs of the tile that are not summed here have no records: their loads return zeros without traffic
    auto bytes_of = [&](u32 t, u32 bytes, bool live) { return live && bpt + t >= bp0 && bpt + t < bp1 ? (int)bytes : 0; };
    const double *wdbl[NP];                                        // unpacked store: pairs beyond the last repeat it
#pragma unroll
    for (u32 t = 0; t < NP; ++t)
        wdbl[t] = reinterpret_cast<const double *>(w) + ((size_t)min(bpt + t, BP - 1) * GQ + 4 * r_first) * w_stride + row;
    // steps 2 g2, 2 g2 + 1 into buffer g2 & 1, with the even one the record's top bits into buffer (g2 / 2) & 1
    auto fetch_w = [&](u32 buf, u32 tbuf, u32 g2) {
        if (PACKED) {
#pragma unroll
            for (u32 t = 0; t < NP; ++t) {
                unsigned char *const at = const_cast<unsigned char *>(wrec) + t * REC_BYTES;
                const __amdgpu_buffer_rsrc_t rs =
                    __builtin_amdgcn_make_buffer_rsrc(at, 0, bytes_of(t, REC_BYTES, true), 0x00020000);
                const u32x4 lo = __builtin_amdgcn_raw_buffer_load_b128(rs, (int)(lane * 16 + buf * 1024), 0, NTW);
                const u32x2 mid = __builtin_amdgcn_raw_buffer_load_b64(rs, (int)(lane * 8 + REC_MID + buf * 512), 0, NTW);
#pragma unroll
                for (u32 z = 0; z < 4; ++z) wr[buf][t][z] = lo[z];
                wr[buf][t][4] = mid[0];
                wr[buf][t][5] = mid[1];
                if (buf == 0)
                    wt[tbuf][t] = __builtin_amdgcn_raw_buffer_load_b32(rs, (int)((lane >> 1) * 4 + REC_TOP), 0, NTW);
            }
            if (buf == 1 && g2 + 1 < 2 * r_end) wrec += wpairs * REC_BYTES;   // the last record stays the last
        } else {
#pragma unroll
            for (u32 t = 0; t < NP; ++t)
#pragma unroll
                for (u32 s = 0; s < 2; ++s) {
                    const bool live = 2 * g2 + s >= gq0 && 2 * g2 + s < gq1;
                    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
                        const_cast<double *>(wdbl[t]), 0, bytes_of(t, N * sizeof(double), live), 0x00020000);
                    const dvec_t v = __builtin_bit_cast(dvec_t, __builtin_amdgcn_raw_buffer_load_b128(rs, (int)(k * 8), 0, 0));
                    wp[s][t][0] = v[0];
                    wp[s][t][1] = v[1];
                    wdbl[t] += w_stride;
                }
        }
    };
    // the weight whose w + 2^49 has the bits hi:lo: 2^52 + (w + 2^49) from its bits, then one exact subtraction
    auto unpack = [](u32 hi, u32 lo) {
        return __hiloint2double((int)(0x43300000u | hi), (int)lo) - (4503599627370496.0 + 562949953421312.0);
    };
    // Step s of two, pairs in order in the first and in reverse in the second: a product needs its sum's old and new
    // high parts at once, and with this order the new one finds its place in the register the previous sum has left,
    // and goes back in the next step, so that no copies are needed.  One pair at a time: the barriers keep the compiler
    // from unpacking all pairs first, which takes more registers than two waves per SIMD have.
    auto products = [&](u32 buf, u32 tbuf, u32 s) {
#pragma unroll
        for (u32 tt = 0; tt < NP; ++tt) {
            const u32 t = s ? NP - 1 - tt : tt;
            double wd[2];
            if (PACKED) {
                u32 top = wt[tbuf][t], mid = wr[buf][t][4 + s];
                asm volatile("" : "+v"(top), "+v"(mid));
                top >>= top_shift;
#pragma unroll
                for (u32 e = 0; e < 2; ++e) {
                    wd[e] = unpack((((top >> (16 * buf + 8 * s + 2 * e)) & 3u) << 16) | (e ? mid >> 16 : mid & 0xffffu),
                                   wr[buf][t][2 * s + e]);
                }
            } else {
                wd[0] = wp[s][t][0];
                wd[1] = wp[s][t][1];
            }
            // weight of k serves k and N-1-k; weight of k+1 serves k+1 and N-2-k
#pragma unroll
            for (u32 oo = 0; oo < 2 * CO; ++oo) {
                const u32 o = s ? 2 * CO - 1 - oo : oo, c = o / CO, e = o % CO;
                a[t][c][e].mac(x[SH ? 0 : s][c][e >> 1][e & 1], wd[e < 2 ? e : 3 - e]);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    auto fold = [&]() {
#pragma unroll
        for (u32 t = 0; t < NP; ++t)
#pragma unroll
            for (u32 c = 0; c < 2; ++c)
#pragma unroll
                for (u32 e = 0; e < CO; ++e) a[t][c][e].fold(q, u);
    };
    // two steps; the next two's weights are on their way before the products
    auto two_steps = [&](u32 buf, u32 tbuf, u32 g2) {
        if (SH) {
            fetch_shared(g2 + 1);
            if (live) {
                fetch_w(buf ^ 1, buf ? tbuf ^ 1 : tbuf, g2 + 1);
                take_shared(buf, 0);
                products(buf, tbuf, 0);
                take_shared(buf, 1);
                products(buf, tbuf, 1);
            }
            keep_shared(buf ^ 1);
            __syncthreads();
            return;
        }
        if (PACKED) fetch_w(buf ^ 1, buf ? tbuf ^ 1 : tbuf, g2 + 1);
        products(buf, tbuf, 0);
        fetch_x(0, 2 * g2 + 2);
        products(buf, tbuf, 1);
        if (!PACKED) fetch_w(0, 0, g2 + 1);
        fetch_x(1, 2 * g2 + 3);
    };
    // whole records of four steps, whatever the range: 8 products between two folds
    if (r_first < r_end) {
        fetch_w(0, 0, 2 * r_first);
        if (SH) {
            fetch_shared(2 * r_first);
            keep_shared(0);
            __syncthreads();
        } else {
            fetch_x(0, 4 * r_first);
            fetch_x(1, 4 * r_first + 1);
        }
    }
    for (u32 r = r_first; r < r_end; r += 2) {
        two_steps(0, 0, 2 * r);
        two_steps(1, 0, 2 * r + 1);
        if (r + 1 < r_end) {
            two_steps(0, 1, 2 * r + 2);
            two_steps(1, 1, 2 * r + 3);
        }
        fold();
    }
    // the up to three steps behind the last whole record: all their loads, then the products
    const u32 s0 = max(gq0, 4 * ps.records());
    if (PACKED && s0 < gq1) {
        dvec_t xs[3][2][HV];
        u32x2 lo[3][NP];
        u32 mid[3][NP], top[3][NP];
#pragma unroll
        for (u32 s = 0; s < 3; ++s) {
            const double *xs_at = bank + (size_t)(s0 + s) * 2 * w_stride + row;
#pragma unroll
            for (u32 c = 0; c < 2; ++c) {
                const __amdgpu_buffer_rsrc_t rs =
                    __builtin_amdgcn_make_buffer_rsrc(const_cast<double *>(xs_at + c * w_stride), 0,
                                                      s0 + s < gq1 ? (int)(N * sizeof(double)) : 0, 0x00020000);
#pragma unroll
                for (u32 h = 0; h < HV; ++h)
                    xs[s][c][h] = __builtin_bit_cast(dvec_t, __builtin_amdgcn_raw_buffer_load_b128(rs, (int)(kk[h] * 8), 0, 0));
            }
            const unsigned char *at = reinterpret_cast<const unsigned char *>(w) + ps.step(bpt, i, chunk, s0 - 4 * ps.records() + s);
#pragma unroll
            for (u32 t = 0; t < NP; ++t) {
                const __amdgpu_buffer_rsrc_t rs =
                    __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned char *>(at) + t * STEP_BYTES, 0,
                                                      bytes_of(t, STEP_BYTES, s0 + s < gq1), 0x00020000);
                lo[s][t] = __builtin_amdgcn_raw_buffer_load_b64(rs, (int)(lane * 8), 0, 0);
                mid[s][t] = __builtin_amdgcn_raw_buffer_load_b32(rs, (int)(lane * 4 + STEP_MID), 0, 0);
                top[s][t] = __builtin_amdgcn_raw_buffer_load_b8(rs, (int)((lane >> 1) + STEP_TOP), 0, 0);
            }
        }
#pragma unroll
        for (u32 s = 0; s < 3; ++s)
            if (s0 + s < gq1) {
#pragma unroll
                for (u32 t = 0; t < NP; ++t) {
                    const u32 hb = top[s][t] >> top_shift;
                    double wd[2];
#pragma unroll
                    for (u32 e = 0; e < 2; ++e)
                        wd[e] = unpack(((hb >> (2 * e)) & 3u) << 16 | (e ? mid[s][t] >> 16 : mid[s][t] & 0xffffu), lo[s][t][e]);
#pragma unroll
                    for (u32 o = 0; o < 2 * CO; ++o) {
                        const u32 c = o / CO, e = o % CO;
                        a[t][c][e].mac(xs[s][c][e >> 1][e & 1], wd[e < 2 ? e : 3 - e]);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        fold();
    }
#pragma unroll
    for (u32 t = 0; t < NP; ++t) {
        if (bpt + t >= bp0 && bpt + t < bp1) {
#pragma unroll
            for (u32 c = 0; c < 2; ++c)
#pragma unroll
                for (u32 h = 0; h < HV; ++h) {
                    vec_t o;
                    o[0] = a[t][c][2 * h].canonical(q, u);
                    o[1] = a[t][c][2 * h + 1].canonical(q, u);
                    vec_t *dst = reinterpret_cast<vec_t *>(acc + ((size_t)(bpt + t) * 2 + c) * w_stride + row + kk[h]);
                    if ((size_t)BP * 2 * w_stride * sizeof(u64) > STREAM_BYTES)
                        __builtin_nontemporal_store(o, dst);       // the bank keeps its place in L2 (8449 -> 8316 us)
                    else
                        *dst = o;
                }
        }
    }
}

// Wavefronts that share a chunk's bank residues, by the store (1: half records, 2: whole limbs) and the tiles of the launch:
// four where at most a third more wavefronts go out than have pairs, two for an even number of tiles of whole limbs that would
// waste more than a fifth by four, 1 (each its own) otherwise, for launches that leave CUs idle, and for whole limbs whose bank
// the Infinity Cache holds.  us, own / two / four, tiles in brackets:
//   half records: 2^16 [18] 8417 / 8027 / 7737, [10] 1649 / 1587 / 1548, [9] 1499 / 1478 / 1442, [7] 1168 / 1174 / 1103, [5] 863 /
//     862 / 903, [3] 1158 / 1192 / 1079, [2] 231 / 229 / 232; 2^15 [6] 266 / 250 / 245, [4] 186 / 172 / 160, [3] 158 / 148 / 132;
//     2^14 [4] 54 / 56 / 47, [3] 49 / 49 / 42; 2^13 [4] (96 workgroups) 12.1 / 14.0 / 13.8.  Two spill registers there.
//   whole limbs: 2^15 [8] 1433 / 1340 / 1341, [7] 1295 / 1248 / 1203, [6] 605 / 556 / 590, [5] 951 / 953 / 1015, [4] 768 / 708 / 715,
//     [3] 625 / 614 / 569; 2^16 [3] 917 / 918 / 865, [2] 667 / 618 / 648; a small bank, 2^14 [6] 63.1 / 65.1 / 65.1, 2^13 [4] 10.8 /
//     13.1 / 12.9.
// Half records of short sums: from 24 steps on, or 12 without idle wavefronts.  A short sum has no loop to hide the first two steps'
// way through LDS in.  us, own / four, steps [tiles] of 24 limbs at 2^16: 2 [6] 172 / 208, 4 214 / 241, 8 321 / 351, 10 377 / 430,
// 14 488 / 524, 18 588 / 630, 22 702 / 744, 24 732 / 729, 26 795 / 803; 8 limbs at 2^16: 6 [3] 53 / 63, 10 [3] 80 / 89, 18 126 / 132, 24
// 163 / 162, 2 [9] 88 / 104, 16 [9] 280 / 278; 24 limbs at 2^14: 2 [9] 66 / 80, 6 120 / 135, 16 [3] 74 / 74, 64 240 / 223; without
// idle wavefronts, 12 limbs at 2^15 [8]: 10 138 / 140, 12 147 / 147, 14 171 / 167, 16 189 / 173, 20 229 / 214, 28 301 / 273.
static u32 share_of(u32 store, u32 tiles, u32 steps, u32 N, u32 n_limbs, bool small_bank) {
    const u32 four = (tiles + 3) / 4 * 4, chunks = N / REC_CHUNK / (store == 1 ? 2 : 1);
    if ((store != 1 && (store != 2 || small_bank)) || tiles < 2 || (u64)(four / 4) * chunks * n_limbs < 256) return 1;
    if (store == 1 && steps < (four == tiles ? 12u : 24u)) return 1;
    if (store == 2 && tiles % 2 == 0 && 5 * four > 6 * tiles) return 2;
    return 3 * four <= 4 * tiles ? 4 : 1;
}

// An input ciphertext as the bank entry of the identity rotation: balanced doubles on primes below 2^50, as it is on
// the others.  blockIdx.y = component * level + limb, two residues per thread
__global__ __launch_bounds__(EW_THREADS) void bank_entry_kernel(const u64 *__restrict__ src, u64 *__restrict__ dst,
                                                                const ModConst *__restrict__ mods, u32 level, u32 N) {
    typedef u64 vec_t __attribute__((ext_vector_type(2)));
    const size_t k = (size_t)blockIdx.y * N + (blockIdx.x * EW_THREADS + threadIdx.x) * 2;
    const u64 q = mods[blockIdx.y < level ? blockIdx.y : blockIdx.y - level].q;
    vec_t v = *reinterpret_cast<const vec_t *>(src + k);
    if ((q >> 50) == 0) {
        v[0] = balanced_bits(v[0], q);
        v[1] = balanced_bits(v[1], q);
    }
    *reinterpret_cast<vec_t *>(dst + k) = v;
}

// dst[z][0 .. words) = src[z * src_stride + 0 .. words), z = blockIdx.z; words is a multiple of 2 * EW_THREADS
__global__ __launch_bounds__(EW_THREADS) void copy_blocks_kernel(u64 *__restrict__ dst, const u64 *__restrict__ src,
                                                                 size_t words, size_t src_stride) {
    typedef u64 vec_t __attribute__((ext_vector_type(2)));
    const size_t k = ((size_t)blockIdx.x * EW_THREADS + threadIdx.x) * 2;
    *reinterpret_cast<vec_t *>(dst + blockIdx.z * words + k) =
        *reinterpret_cast<const vec_t *>(src + blockIdx.z * src_stride + k);
}

// y_b = base_b + the rotated accumulators of block b among the cn items of a batch; item r belongs to block (c0 + r) % B.
// base is y itself from the second batch on.  bias: [B][level][N] added to component 0, or null.  blockIdx.y = component *
// level + limb, blockIdx.z = block; two residues per thread.
__global__ __launch_bounds__(EW_THREADS) void add_rotations_kernel(u64 *y, const u64 *base,
                                                                   size_t base_stride, const u64 *__restrict__ items,
                                                                   const u64 *__restrict__ bias,
                                                                   const ModConst *__restrict__ mods, u32 level, u32 N,
                                                                   u32 b0, u32 B, u32 c0, u32 cn) {
    typedef u64 vec_t __attribute__((ext_vector_type(2)));
    const u32 b = b0 + blockIdx.z;
    const size_t ctw = (size_t)2 * level * N;
    const size_t k = (size_t)blockIdx.y * N + (blockIdx.x * EW_THREADS + threadIdx.x) * 2;
    const u64 q = mods[blockIdx.y < level ? blockIdx.y : blockIdx.y - level].q;
    vec_t v = *reinterpret_cast<const vec_t *>(base + (size_t)b * base_stride + k);
    if (bias && blockIdx.y < level) {
        const vec_t x = *reinterpret_cast<const vec_t *>(bias + (size_t)b * level * N + k);
        v[0] = add_mod(v[0], x[0], q);
        v[1] = add_mod(v[1], x[1], q);
    }
    for (u32 r = (b + B - c0 % B) % B; r < cn; r += B) {
        const vec_t x = *reinterpret_cast<const vec_t *>(items + r * ctw + k);
        v[0] = add_mod(v[0], x[0], q);
        v[1] = add_mod(v[1], x[1], q);
    }
    *reinterpret_cast<vec_t *>(y + (size_t)b * ctw + k) = v;
}

// c0 of block b of y [B][2][level][N] += bias[b]: blockIdx.y = limb, blockIdx.z = output block, two residues per thread
__global__ __launch_bounds__(EW_THREADS) void add_bias_kernel(u64 *__restrict__ y,
                                                              const u64 *__restrict__ bias,
                                                              const ModConst *__restrict__ mods, u32 level, u32 N) {
    typedef u64 vec_t __attribute__((ext_vector_type(2)));
    const u32 k = (blockIdx.x * EW_THREADS + threadIdx.x) * 2, i = blockIdx.y, b = blockIdx.z;
    const u64 q = mods[i].q;
    vec_t *dst = reinterpret_cast<vec_t *>(y + ((size_t)b * 2 * level + i) * N + k);
    const vec_t s = *reinterpret_cast<const vec_t *>(bias + ((size_t)b * level + i) * N + k);
    vec_t v = *dst;
    v[0] = add_mod(v[0], s[0], q);
    v[1] = add_mod(v[1], s[1], q);
    *dst = v;
}

// sym[d] is cleared if polynomial d of the chunk is not fixed by X -> X^-1, i.e. breaks
// c[N-j] == -c[j] for 0 < j < N (which also forces c[N/2] == 0)
__global__ __launch_bounds__(EW_THREADS) void check_real_kernel(const int64_t *__restrict__ coef, u32 *sym, u32 N) {
    const u32 n = blockIdx.x * EW_THREADS + threadIdx.x;
    const int64_t *c = coef + (size_t)blockIdx.y * N;
    if (n == 0) return;
    if (c[N - n] != -c[n]) sym[blockIdx.y] = 0;
}

// Byte offsets within a record of step s (0..3), residue r of its chunk (r even: its pair's): low word, middle half, the
// byte with the top bits of r & ~3 .. r | 3.
__device__ __forceinline__ u32 rec_lo(u32 s, u32 r) { return (s >> 1) * 1024 + (r >> 1) * 16 + (s & 1) * 8 + (r & 1) * 4; }
__device__ __forceinline__ u32 rec_mid(u32 s, u32 r) {
    return REC_MID + (s >> 1) * 512 + (r >> 1) * 8 + (s & 1) * 4 + (r & 1) * 2;
}
__device__ __forceinline__ u32 rec_top(u32 s, u32 r) { return REC_TOP + (r >> 2) * 4 + s; }
// The same from the start of the store, for step gq of pair bp and residue k of limb i, in a record of four or of one.
struct PackedPlace {
    size_t lo, mid, top;
};
__device__ __forceinline__ PackedPlace packed_place(const PackedShape &ps, u32 bp, u32 i, u32 gq, u32 k) {
    const u32 r = k & (REC_CHUNK - 1), g = gq >> 2, s = gq & 3;
    if (g < ps.records()) {
        const size_t at = ps.rec(bp, i, k / REC_CHUNK, g);
        return PackedPlace{at + rec_lo(s, r), at + rec_mid(s, r), at + rec_top(s, r)};
    }
    const size_t at = ps.step(bp, i, k / REC_CHUNK, s);
    return PackedPlace{at + r * 4, at + STEP_MID + r * 2, at + STEP_TOP + (r >> 2)};
}

// Canonical residues below 2^50 of c diagonals, consecutive steps gq0 .. gq0 + c - 1 of pair bp -> packed records of the
// first cnt residues of each limb.  in [c][level][N].  A thread packs four residues of two steps that share a part of a
// record (16-byte and 8-byte stores), or of the one of them that is there: the other is left alone.
// grid: x = 1024 residues, y = (pair of steps of the run) * level + limb
__global__ __launch_bounds__(EW_THREADS) void pack_records_kernel(const u64 *__restrict__ in,
                                                                  unsigned char *__restrict__ out,
                                                                  const ModConst *__restrict__ mods, PackedShape ps,
                                                                  u32 N, u32 cnt, u32 bp, u32 gq0, u32 c) {
    const u32 k = (blockIdx.x * EW_THREADS + threadIdx.x) * 4;
    if (k >= cnt) return;
    const u32 i = blockIdx.y % ps.level, g2 = (gq0 >> 1) + blockIdx.y / ps.level;
    const u64 q = mods[i].q;
    u32 lo[2][4], mid[2][2], top[2];
    bool have[2];
#pragma unroll
    for (u32 s = 0; s < 2; ++s) {
        const u32 gq = 2 * g2 + s;
        have[s] = gq >= gq0 && gq < gq0 + c;
        if (!have[s]) continue;
        const u64 *src = in + ((size_t)(gq - gq0) * ps.level + i) * N + k;
        u32 hi[4];
        top[s] = 0;
#pragma unroll
        for (u32 e = 0; e < 4; ++e) {
            const u64 x = src[e], v = (x > q / 2 ? x - q : x) + (1ull << 49);     // w + 2^49, below 2^50
            lo[s][e] = (u32)v;
            hi[e] = (u32)(v >> 32) & 0xffffu;
            top[s] |= (u32)(v >> 48) << (2 * e);
        }
        mid[s][0] = hi[0] | (hi[1] << 16);
        mid[s][1] = hi[2] | (hi[3] << 16);
    }
    if (have[0] && have[1] && g2 >> 1 < ps.records()) {
        const u32 r = k & (REC_CHUNK - 1), st = (2 * g2) & 3;
        unsigned char *rec = out + ps.rec(bp, i, k / REC_CHUNK, g2 >> 1);
        *reinterpret_cast<uint4 *>(rec + rec_lo(st, r)) = make_uint4(lo[0][0], lo[0][1], lo[1][0], lo[1][1]);
        *reinterpret_cast<uint4 *>(rec + rec_lo(st, r + 2)) = make_uint4(lo[0][2], lo[0][3], lo[1][2], lo[1][3]);
        *reinterpret_cast<uint4 *>(rec + rec_mid(st, r)) = make_uint4(mid[0][0], mid[1][0], mid[0][1], mid[1][1]);
        *reinterpret_cast<unsigned short *>(rec + rec_top(st, r)) = (unsigned short)(top[0] | (top[1] << 8));
        return;
    }
#pragma unroll
    for (u32 s = 0; s < 2; ++s)
        if (have[s]) {
            const PackedPlace a = packed_place(ps, bp, i, 2 * g2 + s, k), b = packed_place(ps, bp, i, 2 * g2 + s, k + 2);
            *reinterpret_cast<uint2 *>(out + a.lo) = make_uint2(lo[s][0], lo[s][1]);
            *reinterpret_cast<uint2 *>(out + b.lo) = make_uint2(lo[s][2], lo[s][3]);
            *reinterpret_cast<u32 *>(out + a.mid) = mid[s][0];
            *reinterpret_cast<u32 *>(out + b.mid) = mid[s][1];
            out[a.top] = (unsigned char)top[s];
        }
}

// steps gq0 .. gq0 + gridDim.y / level - 1 of pair bp: half records -> whole-limb records; residue k of the second half
// is residue N-1-k of the first.  grid: x = 1024 residues, y = step * level + limb
__global__ __launch_bounds__(EW_THREADS) void widen_records_kernel(const unsigned char *__restrict__ in,
                                                                   unsigned char *__restrict__ out, PackedShape half,
                                                                   PackedShape whole, u32 N, u32 bp, u32 gq0) {
    const u32 k = (blockIdx.x * EW_THREADS + threadIdx.x) * 4;
    if (k >= N) return;
    const u32 i = blockIdx.y % half.level, gq = gq0 + blockIdx.y / half.level;
    u32 lo[4], hi[4], top = 0;
#pragma unroll
    for (u32 e = 0; e < 4; ++e) {
        const u32 m = k + e < N / 2 ? k + e : N - 1 - (k + e);
        const PackedPlace a = packed_place(half, bp, i, gq, m);
        lo[e] = *reinterpret_cast<const u32 *>(in + a.lo);
        hi[e] = *reinterpret_cast<const unsigned short *>(in + a.mid);
        top |= ((in[a.top] >> ((m & 3) * 2)) & 3u) << (2 * e);
    }
    const PackedPlace a = packed_place(whole, bp, i, gq, k), b = packed_place(whole, bp, i, gq, k + 2);
    *reinterpret_cast<uint2 *>(out + a.lo) = make_uint2(lo[0], lo[1]);
    *reinterpret_cast<uint2 *>(out + b.lo) = make_uint2(lo[2], lo[3]);
    *reinterpret_cast<u32 *>(out + a.mid) = hi[0] | (hi[1] << 16);
    *reinterpret_cast<u32 *>(out + b.mid) = hi[2] | (hi[3] << 16);
    out[a.top] = (unsigned char)top;
}

__global__ __launch_bounds__(EW_THREADS) void fill_u32_kernel(u32 *p, u32 v, u32 n) {
    const u32 i = blockIdx.x * EW_THREADS + threadIdx.x;
    if (i < n) p[i] = v;
}

// Primes of 50 bits and more: 128-bit lazy sums, flushed after as many products as fit one for the largest modulus.
__global__ __launch_bounds__(MM_THREADS) void diag_mac_int_kernel(const u64 *__restrict__ bank,
                                                                  const u64 *__restrict__ w, u64 *__restrict__ acc,
                                                                  const ModConst *__restrict__ mods, LimbIds limbs,
                                                                  u32 level, u32 N, u32 GQ, u32 BP, u32 flush) {
    const u32 bp0 = blockIdx.x * MM_TB;
    const u32 k = blockIdx.y * MM_THREADS + threadIdx.x;
    const u32 i = limbs.id[blockIdx.z];
    const size_t limb_off = (size_t)i * N + k;
    const size_t w_stride = (size_t)level * N;
    const ModConst m = mods[i];
    u128 a0[MM_TB], a1[MM_TB];
    u64 s0[MM_TB], s1[MM_TB];
#pragma unroll
    for (u32 t = 0; t < MM_TB; ++t) {
        a0[t] = {0, 0};
        a1[t] = {0, 0};
        s0[t] = 0;
        s1[t] = 0;
    }
    u32 pending = 0;
    for (u32 gq = 0; gq < GQ; ++gq) {
        const u64 x0 = bank[((size_t)gq * 2 + 0) * w_stride + limb_off];
        const u64 x1 = bank[((size_t)gq * 2 + 1) * w_stride + limb_off];
#pragma unroll
        for (u32 t = 0; t < MM_TB; ++t) {
            if (bp0 + t < BP) {
                const u64 wv = w[((size_t)(bp0 + t) * GQ + gq) * w_stride + limb_off];
                mac(a0[t], x0, wv);
                mac(a1[t], x1, wv);
            }
        }
        if (++pending == flush) {
#pragma unroll
            for (u32 t = 0; t < MM_TB; ++t) {
                s0[t] = add_mod(s0[t], redc(a0[t], m), m.q);
                s1[t] = add_mod(s1[t], redc(a1[t], m), m.q);
                a0[t] = {0, 0};
                a1[t] = {0, 0};
            }
            pending = 0;
        }
    }
#pragma unroll
    for (u32 t = 0; t < MM_TB; ++t) {
        if (bp0 + t < BP) {
            acc[((size_t)(bp0 + t) * 2 + 0) * w_stride + limb_off] = add_mod(s0[t], redc(a0[t], m), m.q);
            acc[((size_t)(bp0 + t) * 2 + 1) * w_stride + limb_off] = add_mod(s1[t], redc(a1[t], m), m.q);
        }
    }
}

// canonical residues -> the internal form the multiply-accumulate kernels read (rows [rows][N], limb = row % period)
__global__ __launch_bounds__(EW_THREADS) void to_weight_form_kernel(u64 *data, const ModConst *__restrict__ mods,
                                                                    const ModFp *__restrict__ modf, u32 period,
                                                                    u32 N) {
    const u32 n = blockIdx.x * EW_THREADS + threadIdx.x;
    const u32 row = blockIdx.y;
    const u32 limb = row % period;
    const size_t idx = (size_t)row * N + n;
    const u64 x = data[idx];
    if (modf[limb].ok) {
        data[idx] = balanced_bits(x, mods[limb].q);
    } else {
        const ModConst m = mods[limb];
        data[idx] = mont_mul(x, m.r2, m);
    }
}

// ---- rescale on rings of 2^12 .. 2^16 with every active prime below 2^50: three kernels, each reading and writing a
// residue once.  (The plain form below takes six: copy of the dropped limb, two inverse passes, rounding terms, two forward
// passes and the division; a ciphertext product and rescale at 2^15 151 us with it, 136 with these; a bank of 12 at 2^14 with
// rescale 194 and 167.)
//   rescale_intt_kernel:  inverse tile pass of the dropped limb, read where it lies;
//   rescale_mid_kernel:   its column pass, r' = r + floor(q_l/2) mod q_l, the rounding term r' mod q_i - floor(q_l/2) mod
//                         q_i of every remaining limb and the column pass of its forward transform, on tiles of
//                         512 coefficients, 32 threads a row;
//   rescale_tile_kernel:  forward tile pass and (c - NTT(delta)) q_l^-1.
// At N = 2^12 the tile passes are whole transforms, and the last kernel forms the rounding terms it transforms itself.
constexpr u32 RS_TILE = 512;

// grid: x = 4096-residue tiles, y = row
template <u32 RL>
__global__ __launch_bounds__(Tile<RL>::THREADS) void rescale_intt_kernel(const u64 *__restrict__ in, u64 *__restrict__ r,
                                                                   const ModFp *__restrict__ modf,
                                                                   const double *__restrict__ twf_inv, u32 level,
                                                                   u32 logN) {
    __shared__ u64 lds[Tile<RL>::WORDS];
    const u64 *src = in + (((size_t)blockIdx.y * level + level - 1) << logN);
    u64 *dst = r + ((size_t)blockIdx.y << logN);
    auto load = [&](u32 idx) { return src[idx]; };
    auto store = [&](u32 idx, u64 v) { dst[idx] = v; };
    pass_b_body<true, RL>(make_field_fp(modf[level - 1], twf_inv, level - 1, logN), logN, lds, load, store);
}

// grid: x = tiles of 512 coefficients, tsplit times, y = row; out rows [rows][level-1].  tsplit > 1 (few rows): the groups of
// limbs of a tile go to that many workgroups, each of which redoes the dropped limb's column pass
__device__ __forceinline__ double rounding_term(double rp, double hi, double q, double u) { return fma(-rint(rp * u), q, rp) - hi; }
template <u32 LOGR>
__global__ __launch_bounds__(256) void rescale_mid_kernel(const u64 *__restrict__ r, u64 *__restrict__ out,
                                                          const ModFp *__restrict__ modf,
                                                          const ModConst *__restrict__ mods,
                                                          const double *__restrict__ twf_inv,
                                                          const double *__restrict__ twf_fwd, u32 level,
                                                          u32 tsplit) {
    constexpr u32 logN = 12 + LOGR, N = 1u << logN, R = 1u << LOGR, COLS = RS_TILE >> LOGR, PER = COLS / 32;
    __shared__ u64 lds[8 * RS_TILE];
    const u32 tid = threadIdx.x, lane = tid & 31, grp = tid / 32, row = blockIdx.y;
    const u32 c0 = blockIdx.x % (N / RS_TILE) * COLS, tpart = blockIdx.x / (N / RS_TILE);
    const u32 il = level - 1;
    const ModFp ml = modf[il];
    if (grp == 0) {
        const FieldFp f = make_field_fp(ml, twf_inv, il, logN);
        const u64 *src = r + (size_t)row * N;
#pragma unroll
        for (u32 c = 0; c < PER; ++c) {
            const u32 col = lane + 32 * c;
            auto load = [&](u32 at, u32 c_) { return (src + at)[c_]; };
            auto store = [&](u32 at, u32, u64 v) { lds[(at >> 12) * COLS + col] = v; };
            pass_a_body<true, LOGR>(f, c0 + col, load, store);
        }
    }
    __syncthreads();
    const double h = (double)(mods[il].q >> 1);
    double rp[2];
#pragma unroll
    for (u32 e = 0; e < 2; ++e) {
        rp[e] = canonical_double(lds[e * 256 + tid]) + h;
        if (rp[e] >= ml.q) rp[e] -= ml.q;                           // r' = (r + h) mod q_l
    }
    __syncthreads();
    for (u32 i0 = tpart * 8; i0 < il; i0 += tsplit * 8) {
        for (u32 t = 0; t < 8 && i0 + t < il; ++t) {
            const double q = modf[i0 + t].q, u = modf[i0 + t].u, hi = fma(-rint(h * u), q, h);
#pragma unroll
            for (u32 e = 0; e < 2; ++e)
                lds[t * RS_TILE + e * 256 + tid] = (u64)__double_as_longlong(rounding_term(rp[e], hi, q, u));
        }
        __syncthreads();
        if (i0 + grp < il) {
            const u32 i = i0 + grp;
            const FieldFp ff = make_field_fp(modf[i], twf_fwd, i, logN);
            u64 *dst = out + ((size_t)row * il + i) * N;
#pragma unroll
            for (u32 c = 0; c < PER; ++c) {
                const u32 col = lane + 32 * c;
                double v[R];
#pragma unroll
                for (u32 j = 0; j < R; ++j)
                    v[j] = __longlong_as_double((long long)lds[grp * RS_TILE + j * COLS + col]);
                radix_fwd<LOGR>(ff, v, 0, 0);
#pragma unroll
                for (u32 j = 0; j < R; ++j) (dst + j * 4096 + c0)[col] = ff.half(v[j]);
            }
        }
        __syncthreads();
    }
}

// grid: x = 4096-residue tiles, y = limb, z = row; out holds delta after its column pass on entry (N = 2^12: r the dropped
// limb's coefficients)
template <u32 RL>
__global__ __launch_bounds__(Tile<RL>::THREADS) void rescale_tile_kernel(const u64 *__restrict__ in, u64 *out,
                                                                   const u64 *__restrict__ r,
                                                                   const ModFp *__restrict__ modf,
                                                                   const ModConst *__restrict__ mods,
                                                                   const double *__restrict__ twf_fwd,
                                                                   const u64 *__restrict__ qlinv, u32 level, u32 logN) {
    typedef u64 vec_t __attribute__((ext_vector_type(2)));
    typedef Tile<RL> TL;
    __shared__ u64 lds[TL::WORDS];
    const u32 i = blockIdx.y, row = blockIdx.z, tid = threadIdx.x, base = blockIdx.x << 12;
    const u64 *src = in + (((size_t)row * level + i) << logN);
    u64 *dst = out + (((size_t)row * (level - 1) + i) << logN);
    const FieldFp f = make_field_fp(modf[i], twf_fwd, i, logN);
    const double c = canonical_double(mont_mul(qlinv[i], 1, mods[i]));        // q_l^-1 (stored in Montgomery form)
    vec_t x[TL::R / 2];
#pragma unroll
    for (u32 e = 0; e < TL::R / 2; ++e) x[e] = *reinterpret_cast<const vec_t *>(src + base + TL::pair(tid, e));
    u64 raw[TL::R];
    if (logN == 12) {
        const ModFp ml = modf[level - 1];
        const double h = (double)(mods[level - 1].q >> 1), hi = fma(-rint(h * f.u), f.q, h);
#pragma unroll
        for (u32 j = 0; j < TL::R; ++j) {
            double rp = canonical_double(r[(size_t)row * 4096 + Round<RL, 0>::elem(j)]) + h;
            if (rp >= ml.q) rp -= ml.q;
            raw[j] = f.bits(rounding_term(rp, hi, f.q, f.u));
        }
    } else {
#pragma unroll
        for (u32 j = 0; j < TL::R; ++j) raw[j] = dst[base + Round<RL, 0>::elem(j)];
    }
    pass_b_fwd_from_regs<true, RL, true>(f, logN, lds, raw, blockIdx.x);
#pragma unroll
    for (u32 e = 0; e < TL::R / 2; ++e) {
        const u32 loc = TL::pair(tid, e);
#pragma unroll
        for (u32 z = 0; z < 2; ++z)
            x[e][z] = f.out(f.mul(canonical_double(x[e][z]) - __longlong_as_double((long long)lds[TL::slot(loc + z)]), c));
        *reinterpret_cast<vec_t *>(dst + base + loc) = x[e];
    }
}

// ---- rescale, plain form
// delta[pc][i][n] = ((r + h) mod q_l) mod q_i - h mod q_i, r = coefficient-domain last limb, h = floor(q_l/2)
__global__ __launch_bounds__(EW_THREADS) void rescale_delta_kernel(const u64 *__restrict__ r, u64 *__restrict__ out,
                                                                   const ModConst *__restrict__ mods, u32 level,
                                                                   u32 N) {
    const u32 n = blockIdx.x * EW_THREADS + threadIdx.x;
    const u32 pc = blockIdx.y;
    const u64 ql = mods[level - 1].q, h = ql >> 1;
    const u64 rp = add_mod(r[(size_t)pc * N + n], h, ql);
    for (u32 i = 0; i + 1 < level; ++i) {
        const ModConst m = mods[i];
        out[((size_t)pc * (level - 1) + i) * N + n] = sub_mod(reduce_any(rp, m), reduce_any(h, m), m.q);
    }
}

// out[pc][i][k] = (in[pc][i][k] - out[pc][i][k]) * q_l^-1 mod q_i   (out holds NTT(delta) on entry)
__global__ __launch_bounds__(EW_THREADS) void rescale_final_kernel(const u64 *__restrict__ in, u64 *out,
                                                                   const ModConst *__restrict__ mods,
                                                                   const u64 *__restrict__ qlinv, u32 level, u32 N) {
    const u32 k = blockIdx.x * EW_THREADS + threadIdx.x;
    const u32 i = blockIdx.y, pc = blockIdx.z;
    const ModConst m = mods[i];
    const size_t o = ((size_t)pc * (level - 1) + i) * N + k;
    out[o] = mont_mul(sub_mod(in[((size_t)pc * level + i) * N + k], out[o], m.q), qlinv[i], m);
}

// gather rows: dst[pc][n] = src[pc][level-1][n]
__global__ __launch_bounds__(EW_THREADS) void take_last_limb_kernel(const u64 *__restrict__ in, u64 *__restrict__ r,
                                                                    u32 level, u32 N) {
    const u32 n = blockIdx.x * EW_THREADS + threadIdx.x;
    const u32 pc = blockIdx.y;
    r[(size_t)pc * N + n] = in[((size_t)pc * level + level - 1) * N + n];
}

// Arena layout of one ckks_ctpt_matmul call, in words: [key-switch scratch | bank | accumulators | merged sums |
// merged digits].
struct MatmulLayout {
    u32 in_chunk, batch, mg_rots;
    size_t dig_w, tmp_w, ks_w, bank_w, acc_w, u_w, mg_w, yfull_w, t_w;
    size_t total() const { return ks_w + bank_w + acc_w + u_w + mg_w + yfull_w + t_w; }
};

constexpr u32 RESCALE_CHUNK = 64;
static int rescale_rows(ckks_params *P, const u64 *d_in, u32 level, u32 rows, u64 *d_out, u64 *d_r, hipStream_t stream);

constexpr size_t SEPARATE_EXTRA = (size_t)256 << 20;
static MatmulLayout matmul_layout_of(const ckks_params *P, const ckks_weights *w, bool merged, bool rescale, u32 batch) {
    MatmulLayout l;
    const u32 N = P->N, level = w->level, G = w->G, B = w->B_out, N2 = w->N2;
    const size_t ctw = (size_t)2 * level * N;
    l.in_chunk = std::min<u32>(ROT_BATCH, G);                    // inputs decomposed together
    l.batch = batch;                                             // inputs or accumulators decomposed and switched together
    l.dig_w = digits_words(P, level);
    l.tmp_w = (size_t)level * N;
    l.ks_w = l.batch * (l.dig_w + l.tmp_w) + switch_scratch_words(P, level, ROT_BATCH);
    // separate giant step: the rotated accumulators of a batch take the bank's place
    const u64 rotated = merged ? 0 : std::min<u64>(l.batch, (u64)B * (N2 - 1));
    l.bank_w = std::max<size_t>((size_t)G * w->N1, rotated) * ctw;
    l.acc_w = (size_t)B * N2 * ctw;
    l.u_w = merged ? (size_t)B * 2 * (level + P->K) * N : 0;    // extended-basis sums of the giant step
    // merged giant step: the digits of up to MERGE_GROUP rotations of one batch of blocks are held together
    l.mg_rots = merged ? std::min<u32>(MERGE_GROUP, N2 - 1) : 0;
    l.mg_w = (size_t)l.mg_rots * std::min(l.batch, B) * l.dig_w;
    // CKKS_MATMUL_RESCALE: the unrescaled blocks and the dropped limbs in the coefficient domain
    l.yfull_w = rescale ? (size_t)B * ctw : 0;
    l.t_w = rescale ? (size_t)std::max<u32>(l.batch, RESCALE_CHUNK) * 2 * N : 0;
    return l;
}

static MatmulLayout matmul_layout(const ckks_params *P, const ckks_weights *w, bool merged, bool rescale = true) {
    const u32 G = w->G, B = w->B_out, N2 = w->N2;
    merged = merged && N2 > 1;
    u32 batch = std::min<u32>(ROT_BATCH, std::max(G, B));
    if (!merged && N2 > 1) {
        // Separate giant step: rotations of several p share a batch as far as memory allows that is reserved anyway, for the
        // merged order of the same projection or by ckks_params_create (a block's worth always fits: the merged order
        // holds larger sums), and a quarter of it, or 256 MiB, beyond.  One block of
        // 256 columns at 2^16, N1 = 16: 15 rotations in one batch 2.98 ms and 3.5 GiB, in two 3.22 ms and 3.1 GiB, one by one
        // 4.58 ms.  Of 64 columns, N1 = 2: all 31 in one batch 3.85 ms and 5.1 GiB, 13 to a batch 4.01 ms and 3.8 GiB.
        size_t have = std::max(matmul_layout_of(P, w, true, true, batch).total(), P->scratch_floor / sizeof(u64));
        have += std::max(have / 4, SEPARATE_EXTRA / sizeof(u64));
        const u32 most = (u32)std::min<u64>(ROT_BATCH, (u64)B * (N2 - 1));
        while (batch < most && matmul_layout_of(P, w, false, true, batch + 1).total() <= have) ++batch;
    }
    return matmul_layout_of(P, w, merged, rescale, batch);
}

size_t matmul_scratch_words(const ckks_params *P, const ckks_weights *w, bool merged) {
    return matmul_layout(P, w, merged).total();
}

int expand_plain(const ckks_params *P, u32 level, const int64_t *d_coeffs, u32 count, u64 *d_out, bool mont,
                        hipStream_t stream) {
    const u32 N = P->N;
    LimbIds ids;
    for (u32 i = 0; i < level; ++i) ids.id[i] = (uint8_t)i;
    const u32 per = std::max<u32>(1, 16384 / level);
    for (u32 done = 0; done < count; done += per) {
        const u32 c = std::min(per, count - done);
        u64 *o = d_out + (size_t)done * level * N;
        int rc;
        // (the fused pass reads a vector once per limb, so its rows may not lie on the vector)
        if (fast_ring(P) && P->logN <= 16 && !words_overlap(d_coeffs, (size_t)count * N, d_out, (size_t)count * level * N)) {
            const auto kernel = P->logN == 12 ? expand_pass_kernel<0> : P->logN == 13 ? expand_pass_kernel<1>
                              : P->logN == 14 ? expand_pass_kernel<2> : P->logN == 15 ? expand_pass_kernel<3>
                                                                                      : expand_pass_kernel<4>;
            hipLaunchKernelGGL(kernel, dim3(N >> 12, c * level), dim3(NTT_THREADS), 0, stream,
                               d_coeffs + (size_t)done * N, o, P->d_mod, P->d_modf, P->d_tws_fwd, P->d_twf_fwd, P->d_ninvs,
                               level);
            CKKS_LAUNCH_CHECK("expand_pass_kernel");
            P->limb_ntts += (u64)c * level;
            rc = P->logN == 12 ? CKKS_OK : launch_ntt(P, o, ids, level, c * level, false, stream, 2);
        } else {
            hipLaunchKernelGGL(expand_coeffs_kernel, dim3(N / EW_THREADS, c), dim3(EW_THREADS), 0, stream,
                               d_coeffs + (size_t)done * N, o, P->d_mod, level, N);
            CKKS_LAUNCH_CHECK("expand_coeffs_kernel");
            rc = launch_ntt(P, o, ids, level, c * level, false, stream);
        }
        if (rc) return rc;
        if (mont) {
            hipLaunchKernelGGL(to_weight_form_kernel, dim3(N / EW_THREADS, c * level), dim3(EW_THREADS), 0, stream, o,
                               P->d_mod, P->d_modf, level, N);
            CKKS_LAUNCH_CHECK("to_weight_form_kernel");
        }
    }
    return CKKS_OK;
}

}  // namespace ckks

using namespace ckks;

extern "C" {

int ckks_weights_create(const ckks_params_t *P, uint32_t level, uint32_t m, uint32_t C, uint32_t G, uint32_t B_out,
                        uint32_t N1, ckks_weights_t **out) {
    if (!out) {
        set_error("ckks_weights_create: out is null");
        return CKKS_E_INVAL;
    }
    *out = nullptr;
    if (!P) {
        set_error("ckks_weights_create: params is null");
        return CKKS_E_INVAL;
    }
    if (level == 0 || level > P->L) {
        set_error("ckks_weights_create: level %u outside [1,%u]", level, P->L);
        return CKKS_E_LEVEL;
    }
    const u32 n = P->N / 2;
    if (!m || !C || !G || !B_out || !N1 || n % m || (n / m) % C || C % N1) {
        set_error("ckks_weights_create: plan m=%u C=%u G=%u B_out=%u N1=%u does not tile %u slots", m, C, G, B_out, N1,
                  n);
        return CKKS_E_INVAL;
    }
    ckks_weights *w = new ckks_weights();
    w->params = P;
    w->level = level;
    w->m = m;
    w->C = C;
    w->G = G;
    w->B_out = B_out;
    w->N1 = N1;
    w->N2 = C / N1;
    w->block_real.assign((size_t)B_out * G, 1);
    w->block_packed.assign((size_t)B_out * G, 0);
    w->loaded.assign((size_t)B_out * w->N2 * G * N1, 0);
    w->packable = P->N >= 4 * MM_THREADS;
    for (u32 i = 0; i < level; ++i)
        if (P->mod[i] >> 50) w->packable = false;
    // the projection's scratch (bank, accumulators, key-switch workspace) is sized here, in either giant-step
    // order, so that ckks_ctpt_matmul itself neither allocates nor synchronises
    ckks_params *Pm = const_cast<ckks_params *>(P);
    CKKS_HIP(hipDeviceSynchronize());
    int rc = Pm->ensure_scratch(std::max(matmul_scratch_words(P, w, false), matmul_scratch_words(P, w, true)) *
                                    sizeof(u64), nullptr);
    if (rc) {
        delete w;
        return rc;
    }
    *out = w;
    return CKKS_OK;
}

namespace {

constexpr u32 STAGE_DIAGS = 32;

int ensure_full_store(ckks_weights *w) {
    if (w->d_w) return CKKS_OK;
    const size_t words = (size_t)w->B_out * w->N2 * w->G * w->N1 * w->level * w->params->N;
    CKKS_HIP(hipMalloc((void **)&w->d_w, words * sizeof(u64)));
    return CKKS_OK;
}

// whole: the store of whole-limb records (general diagonals) instead of the store of half records (real ones)
int ensure_packed_store(ckks_weights *w, bool whole) {
    const u32 N = w->params->N;
    const size_t bytes = packed_shape(N, w->level, w->G * w->N1, w->B_out * w->N2, whole).bytes();
    if (!whole && !w->d_wp) CKKS_HIP(hipMalloc((void **)&w->d_wp, bytes));
    if (whole && !w->d_wpf) CKKS_HIP(hipMalloc((void **)&w->d_wpf, bytes));
    if (!w->d_stage) CKKS_HIP(hipMalloc((void **)&w->d_stage, (size_t)STAGE_DIAGS * w->level * N * sizeof(u64)));
    return CKKS_OK;
}

// A group (b, g) of half records receives a diagonal that is not real: its diagonals move to the whole-limb store.
int widen_group(ckks_weights *w, u32 b, u32 g, hipStream_t stream) {
    int rc = ensure_packed_store(w, true);
    if (rc) return rc;
    const u32 N = w->params->N, GQ = w->G * w->N1;
    for (u32 p = 0; p < w->N2; ++p) {
        hipLaunchKernelGGL(widen_records_kernel, dim3((N / 4 + EW_THREADS - 1) / EW_THREADS, w->N1 * w->level),
                           dim3(EW_THREADS), 0, stream, w->d_wp, w->d_wpf, packed_shape(N, w->level, GQ, w->B_out * w->N2, false),
                           packed_shape(N, w->level, GQ, w->B_out * w->N2, true), N, b * w->N2 + p, g * w->N1);
        CKKS_LAUNCH_CHECK("widen_records_kernel");
    }
    w->block_packed[(size_t)b * w->G + g] = 2;
    return CKKS_OK;
}

}  // namespace

int ckks_weights_set_diagonals(ckks_weights_t *w, uint32_t first, uint32_t count, const int64_t *d_coeffs,
                               void *stream) {
    if (!w || !d_coeffs) {
        set_error("ckks_weights_set_diagonals: null argument");
        return CKKS_E_INVAL;
    }
    const u64 total = (u64)w->B_out * w->N2 * w->G * w->N1;
    if ((u64)first + count > total) {
        set_error("ckks_weights_set_diagonals: [%u,%u) exceeds %llu diagonals", first, first + count,
                  (unsigned long long)total);
        return CKKS_E_INVAL;
    }
    const ckks_params *P = w->params;
    if (count) {
        // real slot vectors are recognised by their coefficients (c[N-j] = -c[j]); an (output block, input group)
        // pair whose diagonals all pass is read through the palindrome kernel.  One host read per chunk: this call is
        // the offline weight-loading step.
        if (w->flag_cap < count) {
            hipFree(w->d_flag);
            w->d_flag = nullptr;
            CKKS_HIP(hipMalloc((void **)&w->d_flag, count * sizeof(u32)));
            w->flag_cap = count;
        }
        hipLaunchKernelGGL(fill_u32_kernel, dim3((count + EW_THREADS - 1) / EW_THREADS), dim3(EW_THREADS), 0,
                           (hipStream_t)stream, w->d_flag, 1u, count);
        hipLaunchKernelGGL(check_real_kernel, dim3(P->N / EW_THREADS, count), dim3(EW_THREADS), 0, (hipStream_t)stream,
                           d_coeffs, w->d_flag, P->N);
        CKKS_LAUNCH_CHECK("check_real_kernel");
        std::vector<u32> flags(count);
        CKKS_HIP(hipMemcpyAsync(flags.data(), w->d_flag, count * sizeof(u32), hipMemcpyDeviceToHost,
                                (hipStream_t)stream));
        CKKS_HIP(hipStreamSynchronize((hipStream_t)stream));
        const u32 N = P->N, level = w->level, N1 = w->N1, G = w->G;
        // the chunk is stored one (b, p, g) run of baby steps at a time; the kind of store is a property of the
        // (output block, input group) pair: packed half records while the pair has seen real diagonals only,
        // packed whole limbs otherwise (chains with a prime of 50 bits or more keep 8-byte words)
        for (u32 lo = first; lo < first + count;) {
            const u32 run = lo / N1;                                   // (b*N2 + p)*G + g
            const u32 g = run % G, b = run / G / w->N2;
            const u32 hi = std::min<u32>(first + count, (run + 1) * N1);
            const size_t grp = (size_t)b * G + g;
            if (w->N1 > 65535 / level) {
                set_error("ckks_weights_set_diagonals: N1 * level = %u exceeds one launch", w->N1 * level);
                return CKKS_E_INVAL;
            }
            bool all_real = true;
            for (u32 d = lo; d < hi; ++d) all_real = all_real && flags[d - first];
            if (!all_real) w->block_real[grp] = 0;
            int rc;
            if (w->packable) {
                const bool whole = !w->block_real[grp];
                if (whole && w->block_packed[grp] == 1 && (rc = widen_group(w, b, g, (hipStream_t)stream))) return rc;
                if ((rc = ensure_packed_store(w, whole))) return rc;
                w->block_packed[grp] = whole ? 2 : 1;
                unsigned char *store = whole ? w->d_wpf : w->d_wp;
                const u32 cnt = whole ? N : N / 2, step0 = g * N1 - run * N1;      // gq of diagonal d: d + step0
                const PackedShape ps = packed_shape(N, level, G * N1, w->B_out * w->N2, whole);
                for (u32 d = lo; d < hi;) {
                    // pieces end at even steps, so that the two steps of a record are packed together
                    const u32 gq = d + step0, c = std::min(STAGE_DIAGS - (gq & 1), hi - d);
                    rc = expand_plain(P, level, d_coeffs + (size_t)(d - first) * N, c, w->d_stage, false,
                                      (hipStream_t)stream);
                    if (rc) return rc;
                    const u32 recs = ((gq + c + 1) >> 1) - (gq >> 1);
                    hipLaunchKernelGGL(pack_records_kernel, dim3((cnt / 4 + EW_THREADS - 1) / EW_THREADS, recs * level),
                                       dim3(EW_THREADS), 0, (hipStream_t)stream, w->d_stage, store, P->d_mod, ps, N, cnt,
                                       run / G, gq, c);
                    CKKS_LAUNCH_CHECK("pack_records_kernel");
                    d += c;
                }
            } else {
                if ((rc = ensure_full_store(w))) return rc;
                rc = expand_plain(P, level, d_coeffs + (size_t)(lo - first) * N, hi - lo,
                                  w->d_w + (size_t)lo * level * N, true, (hipStream_t)stream);
                if (rc) return rc;
            }
            std::fill(w->loaded.begin() + lo, w->loaded.begin() + hi, (uint8_t)1);
            lo = hi;
        }
    }
    return CKKS_OK;
}

int ckks_weights_set_bias(ckks_weights_t *w, const int64_t *d_bias_coeffs, uint64_t bias_mul, void *stream) {
    if (!w || !d_bias_coeffs) {
        set_error("ckks_weights_set_bias: null argument");
        return CKKS_E_INVAL;
    }
    const ckks_params *P = w->params;
    if (!w->d_bias) CKKS_HIP(hipMalloc((void **)&w->d_bias, (size_t)w->B_out * w->level * P->N * sizeof(u64)));
    int rc = expand_plain(P, w->level, d_bias_coeffs, w->B_out, w->d_bias, false, (hipStream_t)stream);
    if (rc) return rc;
    hipLaunchKernelGGL(scale_rows_kernel, dim3(P->N / EW_THREADS, w->B_out * w->level), dim3(EW_THREADS), 0,
                       (hipStream_t)stream, w->d_bias, P->d_mod, w->level, P->N, bias_mul);
    CKKS_LAUNCH_CHECK("scale_rows_kernel");
    return CKKS_OK;
}

int ckks_weights_load(const ckks_params_t *P, uint32_t level, uint32_t m, uint32_t C, uint32_t G, uint32_t B_out,
                      uint32_t N1, const int64_t *d_coeffs, const int64_t *d_bias_coeffs, uint64_t bias_mul,
                      void *stream, ckks_weights_t **out) {
    if (!d_coeffs || !out) {
        set_error("ckks_weights_load: null argument");
        return CKKS_E_INVAL;
    }
    ckks_weights_t *w = nullptr;
    int rc = ckks_weights_create(P, level, m, C, G, B_out, N1, &w);
    if (rc) return rc;
    const uint64_t total = (uint64_t)B_out * w->N2 * G * N1;
    // in pieces of whole (b, p) runs, so that one call's device-side checks stay small
    const uint32_t piece = G * N1 * std::max<uint32_t>(1u, 4096u / (G * N1));
    for (uint64_t first = 0; first < total && rc == CKKS_OK; first += piece)
        rc = ckks_weights_set_diagonals(w, (uint32_t)first, (uint32_t)std::min<uint64_t>(piece, total - first),
                                        d_coeffs + first * P->N, stream);
    if (rc == CKKS_OK && d_bias_coeffs) rc = ckks_weights_set_bias(w, d_bias_coeffs, bias_mul, stream);
    if (rc) {
        ckks_weights_destroy(w);
        return rc;
    }
    *out = w;
    return CKKS_OK;
}

void ckks_weights_destroy(ckks_weights_t *w) {
    if (!w) return;
    hipFree(w->d_w);
    hipFree(w->d_wp);
    hipFree(w->d_wpf);
    hipFree(w->d_stage);
    hipFree(w->d_bias);
    hipFree(w->d_flag);
    delete w;
}

int ckks_ctpt_matmul(ckks_params_t *P, const ckks_weights_t *w, const uint64_t *d_ct_x,
                     const ckks_gkey_t *const *baby_keys, const ckks_gkey_t *const *giant_keys,
                     const ckks_gkey_t *conj_key, uint32_t flags, uint64_t *d_ct_y, ckks_counters_t *counters,
                     void *stream_) {
    hipStream_t stream = (hipStream_t)stream_;
    if (!P || !w || !d_ct_x || !d_ct_y) {
        set_error("ckks_ctpt_matmul: null argument");
        return CKKS_E_INVAL;
    }
    if (w->params != P) {
        set_error("ckks_ctpt_matmul: weights belong to another parameter set");
        return CKKS_E_INVAL;
    }
    const u32 N = P->N, level = w->level, G = w->G, B = w->B_out, N1 = w->N1, N2 = w->N2, m = w->m;
    if ((N1 > 1 && !baby_keys) || (N2 > 1 && !giant_keys)) {
        set_error("ckks_ctpt_matmul: key list missing (N1=%u, N2=%u)", N1, N2);
        return CKKS_E_NOKEY;
    }
    // every key is checked before any work is enqueued
    std::vector<int32_t> baby_steps(N1), giant_steps(N2);
    for (u32 q = 0; q < N1; ++q) baby_steps[q] = (int32_t)(q * m);
    for (u32 p = 0; p < N2; ++p) giant_steps[p] = (int32_t)(p * N1 * m);
    std::vector<const ckks_gkey_t *> bk(N1, nullptr);
    for (u32 q = 1; q < N1; ++q) {
        u64 g;
        ckks_galois_elt(P, baby_steps[q], &g);
        bk[q] = baby_keys[q - 1];
        if (g != 1 && (!bk[q] || bk[q]->params != P || bk[q]->galois_elt != g)) {
            set_error("ckks_ctpt_matmul: baby key %u missing or for the wrong Galois element", q);
            return bk[q] ? CKKS_E_INVAL : CKKS_E_NOKEY;
        }
    }
    std::vector<u64> giant_g(N2, 1);
    for (u32 p = 1; p < N2; ++p) {
        ckks_galois_elt(P, giant_steps[p], &giant_g[p]);
        const ckks_gkey_t *k = giant_keys[p - 1];
        if (giant_g[p] != 1 && (!k || k->params != P || k->galois_elt != giant_g[p])) {
            set_error("ckks_ctpt_matmul: giant key %u missing or for the wrong Galois element", p);
            return k ? CKKS_E_INVAL : CKKS_E_NOKEY;
        }
    }
    if (conj_key && (conj_key->params != P || conj_key->galois_elt != 2ull * P->N - 1)) {
        set_error("ckks_ctpt_matmul: conj_key is not a key for conjugation");
        return CKKS_E_INVAL;
    }
    if (flags & ~(uint32_t)(CKKS_MATMUL_MERGED_GIANT | CKKS_MATMUL_RESCALE | CKKS_MATMUL_CONJ_PER_ACC)) {
        set_error("ckks_ctpt_matmul: unknown flags 0x%x", flags);
        return CKKS_E_INVAL;
    }
    const bool conj_per_acc = (flags & CKKS_MATMUL_CONJ_PER_ACC) != 0;
    if (conj_per_acc && !conj_key) {
        set_error("ckks_ctpt_matmul: CKKS_MATMUL_CONJ_PER_ACC needs conj_key");
        return CKKS_E_NOKEY;
    }
    for (size_t d = 0; d < w->loaded.size(); ++d)
        if (!w->loaded[d]) {
            set_error("ckks_ctpt_matmul: diagonal %zu of %zu was never loaded (ckks_weights_set_diagonals)", d,
                      w->loaded.size());
            return CKKS_E_INVAL;
        }
    const uint64_t ntt0 = P->limb_ntts;
    const size_t ctw = (size_t)2 * level * N;
    const bool rescale = (flags & CKKS_MATMUL_RESCALE) != 0;
    if (rescale && level < 2) {
        set_error("ckks_ctpt_matmul: CKKS_MATMUL_RESCALE needs weights at level 2 or above");
        return CKKS_E_LEVEL;
    }
    if (words_overlap(d_ct_x, (size_t)G * ctw, d_ct_y, (size_t)B * (rescale ? ctw - 2 * N : ctw))) {
        set_error("ckks_ctpt_matmul: d_ct_y overlaps d_ct_x");
        return CKKS_E_INVAL;
    }
    const u32 BP = B * N2, GQ = G * N1;
    // persistent buffers of this call live behind the key-switch scratch
    const bool merged = (flags & CKKS_MATMUL_MERGED_GIANT) && N2 > 1;
    const MatmulLayout lay = matmul_layout(P, w, merged, rescale);
    const u32 in_chunk = lay.in_chunk, batch = lay.batch, mg_rots = lay.mg_rots;
    const size_t dig_w = lay.dig_w, tmp_w = lay.tmp_w, ks_w = lay.ks_w, bank_w = lay.bank_w, acc_w = lay.acc_w,
                 u_w = lay.u_w;
    int rc = P->ensure_scratch(lay.total() * sizeof(u64), stream);   // reserved by ckks_weights_create: no-op
    if (rc) return rc;
    u64 *d_digits = (u64 *)P->d_scratch, *d_tmp = d_digits + batch * dig_w, *d_work = d_tmp + batch * tmp_w;
    u64 *d_bank = (u64 *)P->d_scratch + ks_w, *d_acc = d_bank + bank_w;
    // with CKKS_MATMUL_RESCALE the blocks are assembled at the input level in scratch and leave one limb shorter
    u64 *d_out_final = d_ct_y;
    u64 *d_yfull = d_acc + acc_w + u_w + lay.mg_w, *d_t = d_yfull + lay.yfull_w;
    if (rescale) d_ct_y = d_yfull;
    // ModDown and rescale of the merged giant step in one pass, where the fused kernels apply
    const bool fused_rescale = rescale && merged && !conj_key && moddown_mid_ok(P, level);

    // 1. baby-step bank: the inputs are decomposed once (hoisting); the switches are issued step by step
    //    with the G inputs of one step next to each other, so that they share the reads of that step's key
    std::vector<u64> baby_g(N1, 1);
    for (u32 q = 1; q < N1; ++q) ckks_galois_elt(P, baby_steps[q], &baby_g[q]);
    for (u32 g0 = 0; g0 < G; g0 += in_chunk) {
        const u32 ng = std::min(in_chunk, G - g0);
        const u64 *c1s[ROT_BATCH];
        for (u32 r = 0; r < ng; ++r) c1s[r] = d_ct_x + (size_t)(g0 + r) * ctw + (size_t)level * N;
        rc = decompose(P, c1s, ng, level, d_digits, d_tmp, stream);
        if (rc) return rc;
        SwitchItem items[ROT_BATCH];
        u32 n_it = 0;
        // the inputs of one step stay in one batch; the steps are spread evenly over the batches they need
        u32 n_rot = 0;
        for (u32 q = 0; q < N1; ++q) n_rot += baby_g[q] != 1;
        const u32 per_max = ROT_BATCH / ng, n_batches = (n_rot + per_max - 1) / per_max;
        const u32 per = n_batches ? (n_rot + n_batches - 1) / n_batches : per_max;
        for (u32 q = 0; q < N1; ++q) {
            if (n_it + ng > per * ng) {
                rc = switch_batch(P, level, items, n_it, d_work, stream);
                if (rc) return rc;
                n_it = 0;
            }
            for (u32 r = 0; r < ng; ++r) {
                const u64 *src = d_ct_x + (size_t)(g0 + r) * ctw;
                u64 *dst = d_bank + ((size_t)(g0 + r) * N1 + q) * ctw;
                if (baby_g[q] == 1) {
                    hipLaunchKernelGGL(bank_entry_kernel, dim3(N / (2 * EW_THREADS), 2 * level), dim3(EW_THREADS), 0,
                                       stream, src, dst, P->d_mod, level, N);
                    CKKS_LAUNCH_CHECK("bank_entry_kernel");
                    continue;
                }
                SwitchItem &it = items[n_it++];
                it.balanced = 1;
                it.digits = d_digits + (size_t)r * dig_w;
                it.c1 = src + (size_t)level * N;
                it.c0 = src;
                it.key = bk[q]->d_key;
                it.dst = dst;
                it.galois_elt = baby_g[q];
                it.add = nullptr;
            }
        }
        rc = switch_batch(P, level, items, n_it, d_work, stream);
        if (rc) return rc;
    }
    // 2. diagonal multiply-accumulate
    u64 maxq = 0;
    for (u32 i = 0; i < level; ++i) maxq = std::max(maxq, P->mod[i]);
    const u32 flush = (u32)std::min<u64>(1u << 30, (~0ull) / maxq);
    if (P->prof_on) {
        while (P->prof_ev.size() < P->prof_used + 2) {
            hipEvent_t ev;
            CKKS_HIP(hipEventCreate(&ev));
            P->prof_ev.push_back(ev);
        }
        CKKS_HIP(hipEventRecord(P->prof_ev[P->prof_used], stream));
    }
    {
        LimbIds fp_limbs, int_limbs;
        u32 n_fp = 0, n_int = 0;
        for (u32 i = 0; i < level; ++i) {
            if ((P->mod[i] >> 50) == 0)
                fp_limbs.id[n_fp++] = (uint8_t)i;
            else
                int_limbs.id[n_int++] = (uint8_t)i;
        }
        const dim3 tiles((BP + MM_TB - 1) / MM_TB, N / MM_THREADS);
        // Runs of output blocks whose input groups have the same kinds of store; within a run, one launch per
        // range of input groups of one kind (real diagonals: palindrome kernel on half records; general ones:
        // whole limbs), the later launches adding onto the accumulators of the earlier ones.  Real packing gives
        // one launch; complexified inputs with an odd last group give a general and a real one.
        auto same_kinds = [&](u32 ba, u32 bb) {
            for (u32 g = 0; g < G; ++g)
                if (w->block_real[(size_t)ba * G + g] != w->block_real[(size_t)bb * G + g] ||
                    w->block_packed[(size_t)ba * G + g] != w->block_packed[(size_t)bb * G + g])
                    return false;
            return true;
        };
        for (u32 b0 = 0; n_fp && b0 < B;) {
            u32 b1 = b0 + 1;
            while (b1 < B && same_kinds(b0, b1)) ++b1;
            const u32 bp0 = b0 * N2, bp1 = b1 * N2, tiles4 = (bp1 + TB - 1) / TB - bp0 / TB;
            const u32 in_tile = tiles4 == 1 ? bp1 - bp0 / TB * TB : TB;     // pairs of a lone tile, from its first one
            const bool few = (size_t)GQ * ctw * sizeof(u64) <= STREAM_BYTES;
            const double *bank = reinterpret_cast<const double *>(d_bank);
            const u32 runs = N / (4 * MM_THREADS), gen_runs = N / MM_THREADS / 2;
            for (u32 g0 = 0; g0 < G;) {
                const size_t grp = (size_t)b0 * G + g0;
                u32 g1 = g0 + 1;
                while (g1 < G && w->block_real[grp + (g1 - g0)] == w->block_real[grp] &&
                       w->block_packed[grp + (g1 - g0)] == w->block_packed[grp])
                    ++g1;
                const u32 q0 = g0 * N1, q1 = g1 * N1, add = g0 ? 1u : 0u;
#define MM_LAUNCH(SYM, PACKED, NP, RUNS, WPTR)                                                                     \
    hipLaunchKernelGGL((diag_mac_kernel<SYM, PACKED, NP>), dim3(tiles4, RUNS, n_fp), dim3(MM_THREADS), 0, stream,  \
                       bank, WPTR, d_acc, P->d_modf, fp_limbs, level, N, GQ, BP, (RUNS) % 8 == 0 ? 1u : 0u, q0,    \
                       q1, add, bp0, bp1)
#define MM_SHARED(SYM, S, RUNS, WPTR)                                                                              \
    hipLaunchKernelGGL((diag_mac_kernel<SYM, true, TB, S>), dim3((tiles4 + S - 1) / S, RUNS, n_fp), dim3(MM_THREADS), 0,     \
                       stream, bank, WPTR, d_acc, P->d_modf, fp_limbs, level, N, GQ, BP, (RUNS) % 8 == 0 ? 1u : 0u, q0, q1,  \
                       add, bp0, bp1)
#define MM_LAUNCH_PAIRS(SYM, RUNS, WPTR)                                                                           \
    do {                                                                                                           \
        if (few && in_tile == 1)                                                                                   \
            MM_LAUNCH(SYM, true, 1, RUNS, WPTR);                                                                   \
        else if (few && in_tile == 2)                                                                              \
            MM_LAUNCH(SYM, true, 2, RUNS, WPTR);                                                                   \
        else                                                                                                       \
            MM_LAUNCH(SYM, true, TB, RUNS, WPTR);                                                                  \
    } while (0)
                const u32 share = share_of(w->block_packed[grp], tiles4, q1 - q0, N, n_fp, few);
                if (w->block_packed[grp] == 1 && share == 4)
                    MM_SHARED(true, 4, N / 256, w->d_wp);
                else if (w->block_packed[grp] == 2 && share == 4)
                    MM_SHARED(false, 4, N / 128, w->d_wpf);
                else if (w->block_packed[grp] == 2 && share == 2)
                    MM_SHARED(false, 2, N / 256, w->d_wpf);
                else if (w->block_packed[grp] == 1)
                    MM_LAUNCH_PAIRS(true, runs, w->d_wp);
                else if (w->block_packed[grp] == 2)
                    MM_LAUNCH_PAIRS(false, gen_runs, w->d_wpf);
                else if (w->block_real[grp] && N >= 4 * MM_THREADS)
                    MM_LAUNCH(true, false, TB, runs, w->d_w);
                else
                    MM_LAUNCH(false, false, TB, gen_runs, w->d_w);
#undef MM_SHARED
#undef MM_LAUNCH_PAIRS
#undef MM_LAUNCH
                g0 = g1;
            }
            b0 = b1;
        }
        if (n_int)
            hipLaunchKernelGGL(diag_mac_int_kernel, dim3(tiles.x, tiles.y, n_int), dim3(MM_THREADS), 0, stream, d_bank,
                               w->d_w, d_acc, P->d_mod, int_limbs, level, N, GQ, BP, flush);
        CKKS_LAUNCH_CHECK("diag_mac_kernel");
    }
    if (P->prof_on) {
        CKKS_HIP(hipEventRecord(P->prof_ev[P->prof_used + 1], stream));
        P->prof_used += 2;
    }
    // 2b. decomplexification in the order Sec. 3.2 displays it: acc_{b,p} += conj(acc_{b,p}) for every accumulator,
    //     before the fold over p.  The switch gathers from its source while it writes, so it goes to the output
    //     area (not yet in use) first.
    if (conj_per_acc) {
        const u32 step = std::min(batch, B);
        for (u32 a0 = 0; a0 < BP; a0 += step) {
            const u32 na = std::min(step, BP - a0);
            SwitchItem items[ROT_BATCH];
            const u64 *c1s[ROT_BATCH];
            for (u32 r = 0; r < na; ++r) c1s[r] = d_acc + (size_t)(a0 + r) * ctw + (size_t)level * N;
            rc = decompose(P, c1s, na, level, d_digits, d_tmp, stream);
            if (rc) return rc;
            for (u32 r = 0; r < na; ++r) {
                items[r].digits = d_digits + (size_t)r * dig_w;
                items[r].c1 = c1s[r];
                items[r].c0 = d_acc + (size_t)(a0 + r) * ctw;
                items[r].key = conj_key->d_key;
                items[r].dst = d_ct_y + (size_t)r * ctw;
                items[r].galois_elt = conj_key->galois_elt;
                items[r].add = nullptr;
                items[r].balanced = 0;
            }
            rc = switch_batch(P, level, items, na, d_work, stream);
            if (rc) return rc;
            hipLaunchKernelGGL(add_rows_kernel, dim3(N / EW_THREADS, na * 2 * level), dim3(EW_THREADS), 0, stream,
                               d_acc + (size_t)a0 * ctw, d_ct_y, P->d_mod, level, N);
            CKKS_LAUNCH_CHECK("add_rows_kernel");
        }
    }
    // 3. giant steps: y_b = acc_{b,0} + sum_p rot(acc_{b,p}).  Where ModDown and rescale are one pass and at least one
    //    rotation needs a key, that pass writes the caller's buffer itself and y_b is assembled where acc_{b,0} lies;
    //    otherwise y_b starts as a copy of acc_{b,0} in the output (or its full-level stand-in).  The plain ModDown can write
    //    elsewhere than it reads as well (`apart`: no copy); a conjugation behind it then adds its source itself.
    std::vector<u32> ps;                                      // giant rotations that are not a full turn
    for (u32 p = 1; p < N2; ++p)
        if (giant_g[p] != 1) ps.push_back(p);
    const bool in_place = fused_rescale && !ps.empty();
    const bool apart = !in_place && merged && !ps.empty() && moddown_mid_ok(P, level);
    const bool conj_after = conj_key && !conj_per_acc;
    u64 *y_base = in_place || apart ? d_acc : d_ct_y;
    const size_t y_stride = in_place || apart ? (size_t)N2 * ctw : ctw;
    const bool batched = !merged && !ps.empty();              // y_b starts in the first batch of rotations
    for (u32 b0 = 0; !in_place && !apart && !batched && b0 < B; b0 += 65535) {
        hipLaunchKernelGGL(copy_blocks_kernel, dim3((u32)(ctw / (2 * EW_THREADS)), 1, std::min<u32>(B - b0, 65535)),
                           dim3(EW_THREADS), 0, stream, d_ct_y + (size_t)b0 * ctw, d_acc + (size_t)b0 * N2 * ctw, ctw,
                           (size_t)N2 * ctw);
        CKKS_LAUNCH_CHECK("copy_blocks_kernel");
    }
    u64 *d_u = d_acc + acc_w, *d_mdig = d_u + u_w;
    if (merged) {
        // rotations that are a full turn are plain additions; the others are grouped: the accumulators of a
        // group are decomposed, then one pass sums their switched forms over the extended basis; one ModDown
        // per block follows
        for (u32 p = 1; p < N2; ++p) {
            if (giant_g[p] != 1) continue;
            for (u32 b = 0; b < B; ++b) {
                hipLaunchKernelGGL(add_rows_kernel, dim3(N / EW_THREADS, 2 * level), dim3(EW_THREADS), 0, stream,
                                   y_base + (size_t)b * y_stride, d_acc + ((size_t)b * N2 + p) * ctw, P->d_mod, level, N);
                CKKS_LAUNCH_CHECK("add_rows_kernel");
            }
        }
        for (u32 b0 = 0; !ps.empty() && b0 < B; b0 += batch) {
            const u32 nb = std::min(batch, B - b0);
            const bool half = merged_from_half(P, level, nb);
            u64 *u_b = d_u + (size_t)b0 * 2 * (level + P->K) * N;
            for (size_t i0 = 0; i0 < ps.size(); i0 += mg_rots) {
                MergedRot rots;
                rots.n_rot = (u32)std::min<size_t>(mg_rots, ps.size() - i0);
                // the group's accumulators, rotation-major, are decomposed in as few launches as the batch size
                // allows (their digits fill d_mdig in the same order); the key-switch scratch is idle until the
                // ModDown and holds the coefficient-domain c1 of a whole batch
                const u32 n_dec = rots.n_rot * nb;
                for (u32 c0 = 0; c0 < n_dec; c0 += ROT_BATCH) {
                    const u32 cn = std::min(ROT_BATCH, n_dec - c0);
                    const u64 *c1s[ROT_BATCH];
                    for (u32 c = 0; c < cn; ++c) {
                        const u32 i = (c0 + c) / nb, r = (c0 + c) % nb;
                        c1s[c] = d_acc + ((size_t)(b0 + r) * N2 + ps[i0 + i]) * ctw + (size_t)level * N;
                    }
                    rc = decompose(P, c1s, cn, level, d_mdig + (size_t)c0 * dig_w, d_work, stream, half);
                    if (rc) return rc;
                }
                for (u32 i = 0; i < rots.n_rot; ++i) {
                    const u32 p = ps[i0 + i];
                    rots.key[i] = giant_keys[p - 1]->d_key;
                    rots.galois_elt[i] = giant_g[p];
                    rots.c0_off[i] = (size_t)p * ctw;
                }
                rc = switch_accumulate_merged(P, level, rots, nb, d_mdig, d_acc + (size_t)b0 * N2 * ctw,
                                              (size_t)N2 * ctw, y_base + (size_t)b0 * y_stride, y_stride, u_b, i0 > 0,
                                              half, stream);
                if (rc) return rc;
            }
            const u64 *zs[ROT_BATCH];
            u64 *outs[ROT_BATCH];
            for (u32 r = 0; r < nb; ++r) {
                u64 *z = y_base + (size_t)(b0 + r) * y_stride;
                zs[r] = z;
                outs[r] = fused_rescale           ? d_out_final + (size_t)(b0 + r) * (ctw - 2 * N)
                        : apart && !conj_after    ? d_ct_y + (size_t)(b0 + r) * ctw
                                                  : z;
            }
            if (fused_rescale)       // the bias before the ModDown: the rescale needs the complete dropped limb
                rc = moddown_rescale(P, level, u_b, zs, w->d_bias ? w->d_bias + (size_t)b0 * level * N : nullptr, outs, nb,
                                     d_work, d_t, stream);
            else
                rc = moddown_add(P, level, u_b, zs, outs, nb, d_work, stream);
            if (rc) return rc;
        }
    }
    // Separate order: each rotation a complete key switch.  The switches of all rotations and blocks go out in batches of
    // lay.batch, rotation-major (neighbours share the key), into the area of the bank, which is free by now, and are
    // summed from there.  (One batch per rotation before, which with few blocks is a chain of small launches: a 64-wide
    // layer at N = 2^12 with 7 rotations of one block took 57 launches and 501 us, now 21 and 158 us.)
    const bool bias_done = batched && !conj_after;            // the last batch adds it
    for (u64 c0 = 0; batched && c0 < (u64)ps.size() * B; c0 += batch) {
        const u32 cn = (u32)std::min<u64>(batch, (u64)ps.size() * B - c0);
        SwitchItem items[ROT_BATCH];
        const u64 *c1s[ROT_BATCH];
        for (u32 r = 0; r < cn; ++r) {
            const u32 p = ps[(c0 + r) / B], b = (u32)((c0 + r) % B);
            const u64 *src = d_acc + ((size_t)b * N2 + p) * ctw;
            c1s[r] = src + (size_t)level * N;
            items[r].digits = d_digits + (size_t)r * dig_w;
            items[r].c1 = c1s[r];
            items[r].c0 = src;
            items[r].key = giant_keys[p - 1]->d_key;
            items[r].dst = d_bank + (size_t)r * ctw;
            items[r].galois_elt = giant_g[p];
            items[r].add = nullptr;
            items[r].balanced = 0;
        }
        rc = decompose(P, c1s, cn, level, d_digits, d_tmp, stream);
        if (rc) return rc;
        rc = switch_batch(P, level, items, cn, d_work, stream);
        if (rc) return rc;
        for (u32 b0 = 0; b0 < B; b0 += 65535) {
            hipLaunchKernelGGL(add_rotations_kernel, dim3(N / (2 * EW_THREADS), 2 * level, std::min<u32>(B - b0, 65535)),
                               dim3(EW_THREADS), 0, stream, d_ct_y, c0 ? d_ct_y : d_acc, c0 ? ctw : (size_t)N2 * ctw,
                               d_bank, bias_done && c0 + batch >= (u64)ps.size() * B ? w->d_bias : nullptr, P->d_mod, level, N, b0,
                               B, (u32)(c0 % B), cn);
            CKKS_LAUNCH_CHECK("add_rotations_kernel");
        }
    }
    for (u32 p = 1; !merged && p < N2; ++p) {
        if (giant_g[p] != 1) continue;                        // a full turn: plain addition
        for (u32 b = 0; b < B; ++b) {
            hipLaunchKernelGGL(add_rows_kernel, dim3(N / EW_THREADS, 2 * level), dim3(EW_THREADS), 0, stream,
                               d_ct_y + (size_t)b * ctw, d_acc + ((size_t)b * N2 + p) * ctw, P->d_mod, level, N);
            CKKS_LAUNCH_CHECK("add_rows_kernel");
        }
    }
    // 3b. decomplexification: y_b += conj(y_b), one key switch per output block.  The switch gathers from
    //     y_b while it writes: where y_b lies apart from its final place, it goes there, y_b added; otherwise to the (now
    //     free) accumulator area first.
    if (conj_after) {
        for (u32 b0 = 0; b0 < B; b0 += batch) {
            const u32 nb = std::min(batch, B - b0);
            SwitchItem items[ROT_BATCH];
            const u64 *c1s[ROT_BATCH];
            for (u32 r = 0; r < nb; ++r) c1s[r] = y_base + (size_t)(b0 + r) * y_stride + (size_t)level * N;
            rc = decompose(P, c1s, nb, level, d_digits, d_tmp, stream);
            if (rc) return rc;
            for (u32 r = 0; r < nb; ++r) {
                items[r].digits = d_digits + (size_t)r * dig_w;
                items[r].c1 = c1s[r];
                items[r].c0 = c1s[r] - (size_t)level * N;
                items[r].key = conj_key->d_key;
                items[r].dst = apart ? d_ct_y + (size_t)(b0 + r) * ctw : d_acc + (size_t)r * ctw;
                items[r].galois_elt = conj_key->galois_elt;
                items[r].add = apart ? items[r].c0 : nullptr;
                items[r].balanced = 0;
            }
            rc = switch_batch(P, level, items, nb, d_work, stream);
            if (rc) return rc;
            if (apart) continue;
            hipLaunchKernelGGL(add_rows_kernel, dim3(N / EW_THREADS, nb * 2 * level), dim3(EW_THREADS), 0, stream,
                               d_ct_y + (size_t)b0 * ctw, d_acc, P->d_mod, level, N);
            CKKS_LAUNCH_CHECK("add_rows_kernel");
        }
    }
    // 4. bias into c0 of every block; 5. rescale, unless the giant step's ModDown already did both
    for (u32 b0 = 0; w->d_bias && !in_place && !bias_done && b0 < B; b0 += 65535) {
        hipLaunchKernelGGL(add_bias_kernel, dim3(N / (2 * EW_THREADS), level, std::min<u32>(B - b0, 65535)), dim3(EW_THREADS), 0,
                           stream, d_ct_y + (size_t)b0 * ctw, w->d_bias + (size_t)b0 * level * N, P->d_mod, level, N);
        CKKS_LAUNCH_CHECK("add_bias_kernel");
    }
    if (rescale && !in_place) {
        for (u32 b0 = 0; b0 < B; b0 += RESCALE_CHUNK) {
            const u32 c = std::min(RESCALE_CHUNK, B - b0);
            rc = rescale_rows(P, d_ct_y + (size_t)b0 * ctw, level, 2 * c, d_out_final + (size_t)b0 * (ctw - 2 * N), d_t,
                              stream);
            if (rc) return rc;
        }
    }
    if (counters) {
        u64 ks = 0;
        for (u32 q = 1; q < N1; ++q) {
            u64 g;
            ckks_galois_elt(P, baby_steps[q], &g);
            ks += (g != 1) ? G : 0;
        }
        for (u32 p = 1; p < N2; ++p) ks += (giant_g[p] != 1) ? B : 0;
        if (conj_key) ks += conj_per_acc ? BP : B;
        counters->key_switches = ks;
        counters->ptmuls = (u64)GQ * BP;
        counters->limb_ntts = P->limb_ntts - ntt0;
    }
    return CKKS_OK;
}

}  // extern "C"

namespace ckks {

// rescale of `rows` polynomials (rows = 2 x ciphertexts): d_in [rows][level][N] -> d_out [rows][level-1][N];
// d_r: rows*N words of scratch (the last limbs in the coefficient domain)
static int rescale_rows(ckks_params *P, const u64 *d_in, u32 level, u32 rows, u64 *d_out, u64 *d_r,
                        hipStream_t stream) {
    const u32 N = P->N;
    bool fused = P->logN >= 12 && P->logN <= 16;
    for (u32 i = 0; i < level; ++i) fused = fused && (P->mod[i] >> 50) == 0;
    if (fused) {
        const u64 *qlinv = P->d_qlinv + (size_t)(level - 1) * P->L;
        const bool wide_in = wide_tiles((u64)(N >> 12) * rows), wide_out = wide_tiles((u64)(N >> 12) * rows * (level - 1));
        hipLaunchKernelGGL(wide_in ? rescale_intt_kernel<WIDE_RL> : rescale_intt_kernel<4>, dim3(N >> 12, rows),
                           dim3(tile_threads(wide_in)), 0, stream, d_in, d_r, P->d_modf,
                           P->d_twf_inv, level, P->logN);
        CKKS_LAUNCH_CHECK("rescale_intt_kernel");
        const auto mid = P->logN == 12 ? nullptr : P->logN == 13 ? rescale_mid_kernel<1>
                       : P->logN == 14 ? rescale_mid_kernel<2> : P->logN == 15 ? rescale_mid_kernel<3>
                                                                               : rescale_mid_kernel<4>;
        // as many workgroups as fill the chip, as for ModDown.  One ciphertext, never split / up to 512 / 768 / 1024 / 2048
        // workgroups, us: 2^16, level 24 37.2 / 34.9 / 33.7 / 33.6 / 33.3, level 12 28.5 and 27.7, 2^15, level 12 20.7 and 19.4;
        // two at 2^15 27.7 and 26.9, six 41.1 / 40.8 / 40.9 / 41.0 / 42.3, four at 2^16 84.5 / 84.7 / 84.3 / 84.4 / 86.5
        const u32 tsplit = std::max<u32>(1, std::min<u32>((level - 1 + 7) / 8, 768 / (N / RS_TILE * rows)));
        if (mid) {
            hipLaunchKernelGGL(mid, dim3(N / RS_TILE * tsplit, rows), dim3(256), 0, stream, d_r, d_out, P->d_modf, P->d_mod,
                               P->d_twf_inv, P->d_twf_fwd, level, tsplit);
            CKKS_LAUNCH_CHECK("rescale_mid_kernel");
        }
        hipLaunchKernelGGL(wide_out ? rescale_tile_kernel<WIDE_RL> : rescale_tile_kernel<4>, dim3(N >> 12, level - 1, rows),
                           dim3(tile_threads(wide_out)), 0, stream, d_in, d_out, d_r,
                           P->d_modf, P->d_mod, P->d_twf_fwd, qlinv, level, P->logN);
        CKKS_LAUNCH_CHECK("rescale_tile_kernel");
        P->limb_ntts += (u64)rows * level;
        return CKKS_OK;
    }
    hipLaunchKernelGGL(take_last_limb_kernel, dim3(N / EW_THREADS, rows), dim3(EW_THREADS), 0, stream, d_in, d_r,
                       level, N);
    CKKS_LAUNCH_CHECK("take_last_limb_kernel");
    LimbIds ids;
    ids.id[0] = (uint8_t)(level - 1);
    int rc = launch_ntt(P, d_r, ids, 1, rows, true, stream);
    if (rc) return rc;
    hipLaunchKernelGGL(rescale_delta_kernel, dim3(N / EW_THREADS, rows), dim3(EW_THREADS), 0, stream, d_r, d_out,
                       P->d_mod, level, N);
    CKKS_LAUNCH_CHECK("rescale_delta_kernel");
    for (u32 i = 0; i + 1 < level; ++i) ids.id[i] = (uint8_t)i;
    rc = launch_ntt(P, d_out, ids, level - 1, rows * (level - 1), false, stream);
    if (rc) return rc;
    hipLaunchKernelGGL(rescale_final_kernel, dim3(N / EW_THREADS, level - 1, rows), dim3(EW_THREADS), 0, stream, d_in,
                       d_out, P->d_mod, P->d_qlinv + (size_t)(level - 1) * P->L, level, N);
    CKKS_LAUNCH_CHECK("rescale_final_kernel");
    return CKKS_OK;
}

// Scratch of ckks_rescale_static: device memory that exists from load time on every GPU the library runs on, so
// that the entry point never allocates.  In host code the array's name is only a stand-in: its device address is
// looked up once per device (static_scratch_ptr) and that pointer is what kernels and copies receive.
constexpr size_t STATIC_SCRATCH_WORDS = (size_t)1 << 20;          // 8 MiB: 16 limb polynomials at N = 2^16
static __device__ __align__(256) u64 scratch[STATIC_SCRATCH_WORDS];
constexpr int MAX_DEVICES = 64;
static u64 *g_static_ptr[MAX_DEVICES] = {};

static int static_scratch_ptr(int device, u64 **out) {
    if (device < 0 || device >= MAX_DEVICES) {
        set_error("ckks_rescale_static: device %d outside [0,%d)", device, MAX_DEVICES);
        return CKKS_E_INVAL;
    }
    if (!g_static_ptr[device]) {
        u64 *ptr = nullptr;
        CKKS_HIP(hipGetSymbolAddress((void **)&ptr, HIP_SYMBOL(scratch)));
        g_static_ptr[device] = ptr;
    }
    *out = g_static_ptr[device];
    return CKKS_OK;
}

}  // namespace ckks

extern "C" {

int ckks_profile_begin(ckks_params_t *P) {
    if (!P) {
        set_error("ckks_profile_begin: params is null");
        return CKKS_E_INVAL;
    }
    P->prof_on = true;
    P->prof_used = 0;
    return CKKS_OK;
}

int ckks_profile_end(ckks_params_t *P, void *stream, double *total_ms, uint32_t *launches) {
    if (!P || !total_ms || !launches) {
        set_error("ckks_profile_end: null argument");
        return CKKS_E_INVAL;
    }
    CKKS_HIP(hipStreamSynchronize((hipStream_t)stream));
    double sum = 0;
    for (size_t i = 0; i + 1 < P->prof_used; i += 2) {
        float ms = 0;
        CKKS_HIP(hipEventElapsedTime(&ms, P->prof_ev[i], P->prof_ev[i + 1]));
        sum += ms;
    }
    *total_ms = sum;
    *launches = (uint32_t)(P->prof_used / 2);
    P->prof_on = false;
    P->prof_used = 0;
    return CKKS_OK;
}

int ckks_rescale(ckks_params_t *P, const uint64_t *d_ct_in, uint32_t level_in, uint32_t n_ct, uint64_t *d_ct_out,
                 void *stream_) {
    hipStream_t stream = (hipStream_t)stream_;
    if (!P || !d_ct_in || !d_ct_out) {
        set_error("ckks_rescale: null argument");
        return CKKS_E_INVAL;
    }
    if (level_in < 2 || level_in > P->L) {
        set_error("ckks_rescale: level %u outside [2,%u]", level_in, P->L);
        return CKKS_E_LEVEL;
    }
    if (n_ct == 0) return CKKS_OK;
    const u32 N = P->N, level = level_in;
    if (words_overlap(d_ct_in, (size_t)n_ct * 2 * level * N, d_ct_out, (size_t)n_ct * 2 * (level - 1) * N)) {
        set_error("ckks_rescale: d_ct_out overlaps d_ct_in");
        return CKKS_E_INVAL;
    }
    // in slices of RESCALE_CHUNK ciphertexts: the scratch need (one limb polynomial per component) stays within what
    // ckks_params_create reserved
    int rc = P->ensure_scratch((size_t)2 * std::min(n_ct, RESCALE_CHUNK) * N * sizeof(u64), stream);
    if (rc) return rc;
    for (u32 done = 0; done < n_ct; done += RESCALE_CHUNK) {
        const u32 c = std::min(RESCALE_CHUNK, n_ct - done);
        rc = rescale_rows(P, d_ct_in + (size_t)done * 2 * level * N, level, 2 * c,
                          d_ct_out + (size_t)done * 2 * (level - 1) * N, (u64 *)P->d_scratch, stream);
        if (rc) return rc;
    }
    return CKKS_OK;
}

int ckks_rescale_static(ckks_params_t *P, const uint64_t *d_ct_in, uint32_t level_in, uint32_t n_ct,
                        uint64_t *d_ct_out, void *stream_) {
    hipStream_t stream = (hipStream_t)stream_;
    if (!P || !d_ct_in || !d_ct_out) {
        set_error("ckks_rescale_static: null argument");
        return CKKS_E_INVAL;
    }
    if (level_in < 2 || level_in > P->L) {
        set_error("ckks_rescale_static: level %u outside [2,%u]", level_in, P->L);
        return CKKS_E_LEVEL;
    }
    if (n_ct == 0) return CKKS_OK;
    const u32 N = P->N, level = level_in;
    if ((size_t)2 * n_ct * N > STATIC_SCRATCH_WORDS) {
        set_error("ckks_rescale_static: %u ciphertexts of N = %u need %zu words of scratch, the static buffer holds %zu "
                  "(use ckks_rescale)", n_ct, N, (size_t)2 * n_ct * N, STATIC_SCRATCH_WORDS);
        return CKKS_E_INVAL;
    }
    if (words_overlap(d_ct_in, (size_t)n_ct * 2 * level * N, d_ct_out, (size_t)n_ct * 2 * (level - 1) * N)) {
        set_error("ckks_rescale_static: d_ct_out overlaps d_ct_in");
        return CKKS_E_INVAL;
    }
    int device = -1;
    CKKS_HIP(hipGetDevice(&device));
    if (device != P->device) {
        set_error("ckks_rescale_static: current device %d is not the parameter set's device %d", device, P->device);
        return CKKS_E_INVAL;
    }
    u64 *d_r = nullptr;
    int rc = static_scratch_ptr(device, &d_r);
    if (rc) return rc;
    // every word of the buffer this call reads is written first, by rescale_intt_kernel or (other rings and chains)
    // take_last_limb_kernel: nothing to clear
    return rescale_rows(P, d_ct_in, level, 2 * n_ct, d_ct_out, d_r, stream);
}

}  // extern "C"
