// Negacyclic NTT / INTT over the RNS limbs.
//
// out[k] = a(psi^(2*bitrev(k)+1)): the transform splits X^(2t) - psi^(2e) into
// (X^t - psi^e)(X^t + psi^e) stage by stage; stage s has 2^s nodes and node i
// uses the twiddle psi^bitrev(2^s + i).  A polynomial of N = 2^16 residues
// (512 KiB) does not fit LDS, so the stages are cut into two passes over HBM:
//   pass A: the first stages.  Elements that interact there share their index
//           modulo N/2^a; global accesses stay runs of consecutive residues.
//   pass B: the remaining stages act inside aligned runs of consecutive
//           residues; a workgroup owns 4096 of them.
// The inverse runs pass B then pass A with Gentleman-Sande butterflies and folds
// N^-1 into the last stage.
//
// Two implementations:
//  * N = 2^12 .. 2^17: every thread keeps 16 residues (pass A of 2^17: 32) in registers and does four stages (radix 16)
//    between exchanges through LDS.  Pass B covers 12 stages (three rounds, two exchanges) on a 4096-residue tile: the
//    whole transform at N = 2^12, all but the first log N - 12 stages above it.
//    Those stages (pass A) pair residues 4096 apart, so a thread that owns a
//    column holds its rows in registers and needs no LDS at all -- which is what
//    lets the base conversions of key switching, which work column by column in the
//    coefficient domain, carry the neighbouring pass A of both transforms.  Limbs whose prime is
//    below 2^50 run their butterflies in fp64: residues, twiddles and the two halves
//    of a product (a*w = h + l exactly, by FMA) are exact integers in doubles, the
//    quotient comes from one multiplication by 1/q, and values stay signed and
//    unreduced for up to four stages (about 10 issue slots per butterfly instead of
//    about 55 for the 64-bit Montgomery butterfly).  Larger primes (the 60-bit
//    special primes) use lazy integer butterflies with quotient-carrying twiddles in the same kernels.
//  * N = 2^10 and 2^11: a plain kernel with one LDS round trip per stage.  (2^13 .. 2^15 and 2^17 ran on it too: 32
//    polynomials of 9 limbs at 2^15 took 155 us in its two launches, 55 us in these two passes.)
#include <algorithm>

#include "ckks_internal.h"
#include "ntt_device.h"

namespace ckks {

constexpr u32 NTT_TILE_LOG = 12;

// strided != 0: pass A layout, local element (x, lo) = (e / LT, e % LT) sits at
//   x * (N >> a) + blockIdx.x * LT + lo   with LT = T >> a.
// strided == 0: pass B layout, local element e sits at blockIdx.x * T + e.
template <bool INV>
__global__ __launch_bounds__(NTT_THREADS) void ntt_pass_kernel(u64 *__restrict__ data,
                                                               const ModConst *__restrict__ mods,
                                                               const u64 *__restrict__ tw,
                                                               const u64 *__restrict__ ninv, LimbIds ids,
                                                               u32 n_limbs, u32 logN, u32 s_lo, u32 s_hi,
                                                               u32 tile_log, u32 strided) {
    extern __shared__ u64 lds[];
    const u32 row = blockIdx.y;
    const u32 limb = ids.id[row % n_limbs];
    if (limb == SKIP_ROW) return;
    const ModConst m = mods[limb];
    const u32 N = 1u << logN, T = 1u << tile_log;
    u64 *poly = data + (size_t)row * N;
    const u64 *twl = tw + (size_t)limb * N;
    const u32 a = s_hi;                       // pass A always covers stages [0, a)
    const u32 lt_log = tile_log - a;          // only meaningful when strided
    const u32 base = blockIdx.x << (strided ? lt_log : tile_log);

    for (u32 e = threadIdx.x; e < T; e += NTT_THREADS) {
        size_t gi = strided ? ((size_t)(e >> lt_log) << (logN - a)) + base + (e & ((1u << lt_log) - 1)) : base + e;
        lds[e] = poly[gi];
    }
    __syncthreads();

    const u32 n_st = s_hi - s_lo;
    for (u32 st = 0; st < n_st; ++st) {
        const u32 s = INV ? s_hi - 1 - st : s_lo + st;
        // local gap between the two legs of a butterfly
        const u32 gap_log = strided ? tile_log - 1 - s : logN - 1 - s;
        const u32 node0 = strided ? 0 : base >> (logN - s);
        for (u32 bf = threadIdx.x; bf < T / 2; bf += NTT_THREADS) {
            const u32 grp = bf >> gap_log, j = bf & ((1u << gap_log) - 1);
            const u32 i0 = (grp << (gap_log + 1)) + j, i1 = i0 + (1u << gap_log);
            const u64 w = twl[(1u << s) + node0 + grp];
            u64 x = lds[i0], y = lds[i1];
            if (!INV) {
                u64 v = mont_mul(y, w, m);
                lds[i0] = add_mod(x, v, m.q);
                lds[i1] = sub_mod(x, v, m.q);
            } else if (s != 0) {
                lds[i0] = add_mod(x, y, m.q);
                lds[i1] = mont_mul(sub_mod(x, y, m.q), w, m);
            } else {
                lds[i0] = mont_mul(add_mod(x, y, m.q), ninv[2 * limb], m);
                lds[i1] = mont_mul(sub_mod(x, y, m.q), ninv[2 * limb + 1], m);
            }
        }
        __syncthreads();
    }

    for (u32 e = threadIdx.x; e < T; e += NTT_THREADS) {
        size_t gi = strided ? ((size_t)(e >> lt_log) << (logN - a)) + base + (e & ((1u << lt_log) - 1)) : base + e;
        poly[gi] = lds[e];
    }
}


// LOGR: 1 .. 5 = pass A of N = 2^(12+LOGR) (its first / last LOGR stages, registers only; a thread takes 16 residues,
// i.e. 16 >> LOGR columns, so that short rows keep as many loads in flight per wavefront as long ones), 0 = pass B (12
// stages in a 4096 tile)
// KINDS: the rows' primes are all below 2^50 (FP_ROWS: fp64 butterflies), all above and none folds (INT_ROWS), all above
// (INT_ROWS + PM_ROWS) or of any kind (ALL_ROWS).  One launch for rows of several kinds at every size: a launch each, the workgroups of
// the other kind returning at once, costs the latency of a workgroup twice where the chip is not full (the digits of one ciphertext at
// level 17 of 24 + 8 primes 17 + 25 us) and its last waves twice where it is, and the union of the register budgets (pass B 90
// and 98, against 72 and 70 of the fp64 butterflies) keeps the wavefronts that the LDS tile admits.  Two launches and one,
// transform of 50- and 60-bit rows, forward, us: 4096 workgroups at 2^16 112 / 105, 26624 650 / 629, 2560 at 2^15 78 / 63,
// 10240 279 / 251, 2560 and 12800 at 2^14 103 / 68 and 513 / 333, 16000 at 2^13 683 / 418, 3072 at 2^17 93 / 83; inverse alike.
// Rows that do not fold on their own: beside the folding butterflies their tile pass takes 90 registers for 70, a whole forward
// transform of 26 limbs of 61 bits, 30 at a time, at 2^13 61.9 us for 60.5, at 2^14 118 for 115.  Of the other mixtures none gains
// by a kernel of its own (rows that all fold, fp64 and folding, fp64 and quotients: within 1 % at 1, 5 and 30 polynomials).
constexpr int FP_ROWS = 1, INT_ROWS = 2, PM_ROWS = 4, ALL_ROWS = 7;
// + STREAMED: residues go past the caches' replacement order (arrays above STREAM_BYTES): a pass uses each once, and the
// twiddles, as many bytes as a tile and shared by the rows of a limb, stay in L2.  64 x 24 rows at 2^16: tile pass 409 ->
// 383 us, column pass 273 -> 250.  Below that the next pass finds them there: 25 x 14 rows at 2^16 164 us, streamed 182.
constexpr int STREAMED = 8;
constexpr int WIDE = 16;                     // + WIDE: tiles by 1024 threads (pass B only)
// WAVES per SIMD of pass A at 2^17, forward: the butterflies of three kinds of primes take 170 registers, 168 leave a third
// wavefront (two to four constants spilled).  us with two and three: 8 rows of 60-bit primes, batches of 5 / 12, 47.2 / 92.8 and
// 42.7 / 90.4, of 61 and 60 bits, 5: 58.3 and 55.2; batches of 1 to 3 up to 2 % the other way.  Inverse (171) it gains as much
// at a batch of 5 and loses as much at 1.
template <bool INV, u32 LOGR>
constexpr u32 WAVES = LOGR == 5 && !INV ? 3 : 1;
template <bool INV, u32 LOGR, int KIND_NT>
__global__ __launch_bounds__((KIND_NT & WIDE) != 0 ? Tile<WIDE_RL>::THREADS : NTT_THREADS, (WAVES<INV, LOGR>))
void ntt_fast_kernel(u64 *__restrict__ data,
                     const ModConst *__restrict__ mods,
                     const ModFp *__restrict__ modf,
                     const u64 *__restrict__ tw,
                     const double *__restrict__ twf,
                     const u64 *__restrict__ ninv, LimbIds ids,
                     u32 n_limbs, u32 logN) {
    constexpr int KINDS = KIND_NT & ALL_ROWS;
    constexpr bool NT = (KIND_NT & STREAMED) != 0;
    constexpr u32 RL = (KIND_NT & WIDE) != 0 ? WIDE_RL : 4;
    __shared__ u64 lds[LOGR ? 1 : Tile<RL>::WORDS];
    const u32 row = (KINDS & FP_ROWS) && KINDS != FP_ROWS ? gridDim.y - 1 - blockIdx.y : blockIdx.y;   // special limbs come last: start with them
    const u32 limb = ids.id[row - uniform_div(row, n_limbs) * n_limbs];
    if (limb == SKIP_ROW) return;
    const ModFp mf = modf[limb];
    u64 *poly = data + ((size_t)row << logN);
    auto load = [&](u32 idx) { return NT ? __builtin_nontemporal_load(poly + idx) : poly[idx]; };
    auto store = [&](u32 idx, u64 v) {
        if (NT)
            __builtin_nontemporal_store(v, poly + idx);
        else
            poly[idx] = v;
    };
    // (addresses formed per row: with a scalar part the compiler takes 98 registers for 70 here)
    auto load_a = [&](u32 at, u32 col) { return load(at + col); };
    auto store_a = [&](u32 at, u32 col, u64 v) { store(at + col, v); };
    auto go = [&](const auto &f) {
        if constexpr (LOGR == 0) {
            pass_b_body<INV, RL>(f, logN, lds, load, store);
        } else {
            constexpr u32 COLS = LOGR < 4 ? 16u >> LOGR : 1;     // columns of a thread
#pragma unroll
            for (u32 c = 0; c < COLS; ++c)
                pass_a_body<INV, LOGR>(f, (c * gridDim.x + blockIdx.x) * NTT_THREADS + threadIdx.x, load_a, store_a);
        }
    };
    if ((KINDS & FP_ROWS) && (KINDS == FP_ROWS || mf.ok))
        go(make_field_fp(mf, twf, limb, logN));
    else if ((KINDS & PM_ROWS) && (!(KINDS & INT_ROWS) || mf.pm))
        go(make_field_pm(mods, tw, ninv, limb, logN));
    else if (KINDS & INT_ROWS)
        go(make_field_int(mods, tw, ninv, limb, logN));
}

template <bool INV, u32 LOGR>
static void launch_fast(const ckks_params *p, u64 *d_data, const LimbIds &ids, u32 n_limbs, u32 rows,
                        hipStream_t stream, bool scaled_dn) {
    int kinds = 0;
    for (u32 i = 0; i < n_limbs; ++i) {
        if (ids.id[i] == SKIP_ROW) continue;
        const u64 q = p->mod[ids.id[i]];
        kinds |= (q >> 50) == 0 ? FP_ROWS : folds(q) ? PM_ROWS : INT_ROWS;
    }
    const u32 blocks = LOGR == 0 ? p->N >> 12 : LOGR < 4 ? 1u << LOGR : 16;
#define FAST_LAUNCH(KIND)                                                                                            \
    hipLaunchKernelGGL((ntt_fast_kernel<INV, LOGR, KIND>), dim3(blocks, rows), dim3(tile_threads((KIND) & WIDE)), 0, stream, d_data,   \
                       p->d_mod, scaled_dn ? p->d_modf_dn : p->d_modf, INV ? p->d_tws_inv : p->d_tws_fwd,            \
                       INV ? p->d_twf_inv : p->d_twf_fwd, scaled_dn ? p->d_ninvs_dn : p->d_ninvs, ids, n_limbs,      \
                       p->logN)
#define FAST_LAUNCH_KIND(F)                                                                                          \
    do {                                                                                                             \
        switch (kinds) {                                                                                             \
            case FP_ROWS: FAST_LAUNCH(FP_ROWS + (F)); break;                                                         \
            case INT_ROWS: FAST_LAUNCH(INT_ROWS + (F)); break;                                                       \
            case 0: break;                                                                                           \
            case PM_ROWS:                                                                                            \
            case INT_ROWS + PM_ROWS: FAST_LAUNCH(INT_ROWS + PM_ROWS + (F)); break;                                   \
            default: FAST_LAUNCH(ALL_ROWS + (F));                                                                    \
        }                                                                                                            \
    } while (0)
    constexpr int W = LOGR == 0 ? WIDE : 0;
    if (LOGR == 0 && wide_tiles((u64)blocks * rows))
        FAST_LAUNCH_KIND(W);
    else if ((u64)rows * p->N * sizeof(u64) > STREAM_BYTES)
        FAST_LAUNCH_KIND(STREAMED);
    else
        FAST_LAUNCH_KIND(0);
#undef FAST_LAUNCH_KIND
#undef FAST_LAUNCH
}

// pass A of a ring above 2^12
template <bool INV>
static void launch_pass_a(const ckks_params *p, u64 *d_data, const LimbIds &ids, u32 n_limbs, u32 rows,
                          hipStream_t stream, bool scaled_dn) {
    switch (p->logN) {
        case 13: launch_fast<INV, 1>(p, d_data, ids, n_limbs, rows, stream, scaled_dn); break;
        case 14: launch_fast<INV, 2>(p, d_data, ids, n_limbs, rows, stream, scaled_dn); break;
        case 15: launch_fast<INV, 3>(p, d_data, ids, n_limbs, rows, stream, scaled_dn); break;
        case 16: launch_fast<INV, 4>(p, d_data, ids, n_limbs, rows, stream, scaled_dn); break;
        case 17: launch_fast<INV, 5>(p, d_data, ids, n_limbs, rows, stream, scaled_dn); break;
    }
}

int launch_ntt(const ckks_params *p, u64 *d_data, const LimbIds &ids, u32 n_limbs, u32 rows, bool inverse,
               hipStream_t stream, u32 pass_mask, bool scaled_dn) {
    if (rows == 0) return CKKS_OK;
    const u32 logN = p->logN;
    const u32 tile_log = logN < NTT_TILE_LOG ? logN : NTT_TILE_LOG;
    const u32 a = logN > NTT_TILE_LOG ? logN - 8 : 0;
    const size_t lds_bytes = sizeof(u64) << tile_log;
    dim3 grid(p->N >> tile_log, rows), block(NTT_THREADS);
    if (pass_mask & 1)
        for (u32 r = 0; r < rows; ++r)
            if (ids.id[r % n_limbs] != SKIP_ROW) ++p->limb_ntts;
    if (rows > 65535) {
        set_error("launch_ntt: %u rows exceed one launch", rows);
        return CKKS_E_INVAL;
    }
    if (fast_ring(p)) {
        // pass A (log N - 12 stages) and pass B (12 stages); N = 2^12: pass B is the whole transform (forward: the
        // "second" pass, inverse: the "first"), and carries the scaled last stage
        const bool two = logN != 12;
        if (!inverse) {
            if ((pass_mask & 1) && two) launch_pass_a<false>(p, d_data, ids, n_limbs, rows, stream, false);
            if (pass_mask & 2) launch_fast<false, 0>(p, d_data, ids, n_limbs, rows, stream, false);
        } else {
            if (pass_mask & 1) launch_fast<true, 0>(p, d_data, ids, n_limbs, rows, stream, two ? false : scaled_dn);
            if ((pass_mask & 2) && two) launch_pass_a<true>(p, d_data, ids, n_limbs, rows, stream, scaled_dn);
        }
        CKKS_LAUNCH_CHECK("ntt_fast_kernel");
        return CKKS_OK;
    }
    const u64 *ninv_tab = scaled_dn ? p->d_ninv_dn : p->d_ninv;
    if (!inverse) {
        if (a)
            hipLaunchKernelGGL(ntt_pass_kernel<false>, grid, block, lds_bytes, stream, d_data, p->d_mod, p->d_tw_fwd,
                               p->d_ninv, ids, n_limbs, logN, 0u, a, tile_log, 1u);
        hipLaunchKernelGGL(ntt_pass_kernel<false>, grid, block, lds_bytes, stream, d_data, p->d_mod, p->d_tw_fwd,
                           p->d_ninv, ids, n_limbs, logN, a, logN, tile_log, 0u);
    } else {
        hipLaunchKernelGGL(ntt_pass_kernel<true>, grid, block, lds_bytes, stream, d_data, p->d_mod, p->d_tw_inv,
                           ninv_tab, ids, n_limbs, logN, a, logN, tile_log, 0u);
        if (a)
            hipLaunchKernelGGL(ntt_pass_kernel<true>, grid, block, lds_bytes, stream, d_data, p->d_mod, p->d_tw_inv,
                               ninv_tab, ids, n_limbs, logN, 0u, a, tile_log, 1u);
    }
    CKKS_LAUNCH_CHECK("ntt_pass_kernel");
    return CKKS_OK;
}

}  // namespace ckks

using namespace ckks;

static int ntt_api(const ckks_params_t *P, uint64_t *d_data, const uint32_t *limb_ids, uint32_t n_limbs,
                   uint32_t batch, void *stream, bool inverse) {
    if (P && batch == 0) return CKKS_OK;
    if (!P || !d_data || !limb_ids || n_limbs == 0 || n_limbs > MAX_LIMBS) {
        set_error("ckks_ntt: null argument or n_limbs outside [1,%u]", MAX_LIMBS);
        return CKKS_E_INVAL;
    }
    LimbIds ids;
    for (u32 i = 0; i < n_limbs; ++i) {
        if (limb_ids[i] >= P->W) {
            set_error("ckks_ntt: limb id %u out of range", limb_ids[i]);
            return CKKS_E_INVAL;
        }
        ids.id[i] = (uint8_t)limb_ids[i];
    }
    // long batches go out in slices of at most 32768 rows
    u32 per = (32768 / n_limbs) * n_limbs;
    for (u64 done = 0; done < (u64)batch * n_limbs; done += per) {
        u32 rows = (u32)std::min<u64>(per, (u64)batch * n_limbs - done);
        int rc = launch_ntt(P, d_data + done * P->N, ids, n_limbs, rows, inverse, (hipStream_t)stream);
        if (rc) return rc;
    }
    return CKKS_OK;
}

extern "C" {

int ckks_ntt(const ckks_params_t *P, uint64_t *d_data, const uint32_t *limb_ids, uint32_t n_limbs, uint32_t batch,
             void *stream) {
    return ntt_api(P, d_data, limb_ids, n_limbs, batch, stream, false);
}

int ckks_intt(const ckks_params_t *P, uint64_t *d_data, const uint32_t *limb_ids, uint32_t n_limbs, uint32_t batch,
              void *stream) {
    return ntt_api(P, d_data, limb_ids, n_limbs, batch, stream, true);
}

}  // extern "C"
