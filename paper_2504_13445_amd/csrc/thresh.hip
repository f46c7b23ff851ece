// Stage (a): tau_u, the k-th largest u . p over all items (Def. 1), exact.
//
// Screening.  A workgroup holds 32 users per wave in registers and streams the
// items in descending-norm order (Alg. 1 step (1)), 64 per tile, through
// the matrix cores in FP32 (as two FP16 parts from d = 32 on), BF16 or FP8
// (e4m3), with a power-of-two scale per user and per item tile where the
// format needs one.  With N = ||x||, Nh = ||xq|| and R = ||x - xq||
// of the quantized copies xq (all rounded up), every screened value vh
// satisfies |vh - v| <= E(u, p) = R_u N_p + Nh_u R_p + c Nh_u Nh_p +
// c2 N_u N_p + e_abs against the exact value v: the quantisation error by
// Cauchy-Schwarz, c bounds the matrix-core accumulation, c2 the FP64
// definition's own rounding and the FP32 comparisons.
//
// Phase 1 (first t0 tiles): per lane and register slot the running maximum
// of the lower bounds vh - E; the k-th largest of the 64 slot maxima of a
// user (each slot covers a distinct set of items) is a value L0 that at
// least k items reach, so L0 <= tau_u.
// Phase 2 (all tiles, interleaved over `nsplit` workgroups): an item is a
// candidate when vh + E >= L0; S_k(u) lies among the candidates because
// v >= tau_u >= L0.  A tile whose largest norm satisfies
// N_u * N_p * (1 + 2 c) < L0 for every user of the workgroup ends the scan:
// by Cauchy-Schwarz (Eq. 2) no later item can be a candidate (the early stop
// of the paper's norm-ordered scan, Sec. 4.2); the quantisation terms enter
// through the largest ratio over the tiles of a tile's largest R and largest N
// (by tiles, because an item far smaller than its tile's largest, whose scale
// it shares, has R_p / N_p near 1, and K_u would triple for every user: 100k x
// 20k x 64, k = 10, FP32, three items of 1e-10 of their norm: 1.90e9 pairs
// scanned by items, 0.85e9 by tiles, as without them).
// Final: per user, L* = k-th largest lower bound among the candidates (the
// candidates hold every item whose lower bound reaches L0, so this is the
// k-th largest over all items), the candidates with vh + E >= L* are
// recomputed in FP64, and the k-th in (value desc, id asc) order is tau_u.
// A user whose candidates overflow the list is recomputed by brute force.
#include "common.h"
#include "kernels.h"

namespace rmips {


// Bitonic sort of 32 registers, descending.
__device__ __forceinline__ void cas_desc(float &a, float &b) {
    float hi = fmaxf(a, b), lo = fminf(a, b);
    a = hi;
    b = lo;
}

__device__ __forceinline__ void sort32_desc(float (&v)[32]) {
#pragma unroll
    for (int k = 2; k <= 32; k <<= 1) {
#pragma unroll
        for (int j = k >> 1; j > 0; j >>= 1) {
#pragma unroll
            for (int i = 0; i < 32; ++i) {
                int l = i ^ j;
                if (l > i) {
                    if ((i & k) == 0) cas_desc(v[i], v[l]);
                    else cas_desc(v[l], v[i]);
                }
            }
        }
    }
}

// Sort a bitonic sequence of 32 registers, descending.
__device__ __forceinline__ void merge32_desc(float (&v)[32]) {
#pragma unroll
    for (int j = 16; j > 0; j >>= 1) {
#pragma unroll
        for (int i = 0; i < 32; ++i) {
            int l = i ^ j;
            if (l > i) cas_desc(v[i], v[l]);
        }
    }
}

// Screening configuration: up to 12 waves of 32 users (the users' rows stay
// in registers), two item-tile buffers in LDS (the next tile is copied in while
// the current one is used; the registers allow one workgroup per CU, which
// has the LDS to itself), nch 16-byte chunks per half row.
// 12 waves while a half row fits in 8 chunks, or 14 in BF16 (three waves
// per SIMD, 168 registers each; longer rows would spill), 8 up
// to 28 chunks (two per SIMD, 256 registers each: a wave's band test then
// runs while the other wave of its SIMD multiplies), 4 for longer rows,
// whose waves need more registers
__host__ __device__ constexpr int screen_waves(int prec, int nch) {
    return (nch <= 8 || (prec == PREC_BF16 && nch <= 14)) ? 12 : nch <= 28 ? 8 : 4;
}
// the bounds-only pass (phase 1 alone, fewer registers): 8 waves, two
// workgroups per CU (128 registers) while a half row fits in 8 chunks
__host__ __device__ constexpr int screen_waves_p1(int prec, int nch) {
    return nch <= 8 ? 8 : screen_waves(prec, nch);
}
template <bool LISTED> __host__ __device__ constexpr int screen_nw(int prec, int nch) {
    return LISTED ? screen_waves(prec, nch) : screen_waves_p1(prec, nch);
}
template <bool LISTED> __host__ __device__ constexpr int screen_wpe(int prec, int nch) {
    return (!LISTED && nch <= 8) ? 4 : screen_waves(prec, nch) / 4;
}
// per tile buffer: N, Nh, R of the 64 items, the tile's largest Nh and R
// and its scale in the first three of 64 slots, and the items' caller ids
// (copied in with the tile, so that no global load is waited for)
constexpr int NSTRIDE = 5 * TILE_ITEMS;
size_t thresh_screen_lds(int prec, int D) {
    const int ls = lds_row_bytes(prec, D);
    return 2 * (size_t)(TILE_ITEMS * ls + LDS_GUARD) + 2 * (size_t)NSTRIDE * 4 +
           16 * sizeof(float);
}

// Item tile t (64 rows, and per item N, Nh, R, and the tile's scalars) into
// LDS buffer b by direct copies; the last wave also takes the per-item
// arrays.  Completion: dma_wait() and a barrier.
template <int NW>
__device__ __forceinline__ void tile_copy(const ThreshArgs &a, int t, int rowb, int w16,
                                          uint32_t magic, int ls, uint8_t *Pbase, float *Nbase,
                                          int b, int w, int lane) {
    const int64_t rb = (int64_t)t * TILE_ITEMS;
    rows_dma(reinterpret_cast<const uint8_t *>(a.Pq) + rb * rowb, rowb, w16, magic,
             TILE_ITEMS - 1, Pbase + (size_t)b * (TILE_ITEMS * ls + LDS_GUARD), w, NW, lane);
    if (w == NW - 1) {
        float *nb = Nbase + b * NSTRIDE;
        dma4(a.Np + rb + lane, nb);
        dma4(a.Nhp + rb + lane, nb + TILE_ITEMS);
        dma4(a.Rp + rb + lane, nb + 2 * TILE_ITEMS);
        const float *sc = lane == 1 ? a.tmax_r + t : (lane == 2 ? a.sp + rb : a.tmax_nh + t);
        dma4(sc, nb + 3 * TILE_ITEMS);
        const int64_t pr = rb + lane < a.m ? rb + lane : a.m - 1;  // padding rows: never candidates
        dma4(a.perm + pr, nb + 4 * TILE_ITEMS);
    }
}

// Element i (0..31) of the pair of accumulators (register i & 15 of block
// i >> 4) for a per-lane i, by selects (no dynamic register index).
__device__ __forceinline__ float pick32(const f32x16 &a0, const f32x16 &a1, int i) {
    const int j = i & 15;
    float x = a0[0], y = a1[0];
#pragma unroll
    for (int q = 1; q < 16; ++q) {
        x = (j == q) ? a0[q] : x;
        y = (j == q) ? a1[q] : y;
    }
    return (i & 16) ? y : x;
}

// Users of one screening workgroup: 32 per wave.  Without a user list the
// grid covers all users once; with one (refinement passes) the workgroups
// stride over the list, whose length is read on the device.
__device__ __forceinline__ int64_t screen_blocks(const ThreshArgs &a, int tu) {
    const int64_t cnt = a.ulist ? (int64_t)*a.ulist_cnt : a.n;
    return (cnt + tu - 1) / tu;
}

// LISTED: a pass over a user list (its own kernel symbol).  What bounds it is
// the matrix cores: split FP32 rows take 6 products of 64 x 32 values per 16
// terms from 4 LDS reads, 1.27 PFLOP/s of FP16 products at 2,000,000 users x
// 28,000 scanned items x 200 (55 ms; FP32 matrix steps took 173 ms, 0.82 of
// their peak).
template <int PREC, int NCH, bool LISTED>
// three, two or one waves per SIMD, as the wave count above sets
__global__ __launch_bounds__(64 * screen_nw<LISTED>(PREC, NCH)) __attribute__((amdgpu_waves_per_eu(screen_wpe<LISTED>(PREC, NCH))))
void k_thresh_screen(ThreshArgs a) {
    constexpr int NW = screen_nw<LISTED>(PREC, NCH), TU = 32 * NW;
    extern __shared__ __align__(16) uint8_t smem8[];
    const int D = a.D, ls = lds_row_bytes(PREC, D), rowb = D * elem_bytes(PREC);
    const int nch = rowb / 32;
    // item tiles, each followed by LDS_GUARD bytes of zeros; then N, Nh, R
    const int bstride = TILE_ITEMS * ls + LDS_GUARD;
    uint8_t *Pbase = smem8;
    float *Nbase = reinterpret_cast<float *>(Pbase + 2 * bstride);
    float *red = reinterpret_cast<float *>(Nbase + 2 * NSTRIDE);

    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int split = blockIdx.y;
    const int w16 = rowb / 16;
    const int ucol = w * 32 + (lane & 31);
    constexpr bool listed = LISTED;
    const int64_t nlist = listed ? (int64_t)*a.ulist_cnt : a.n;
    const int64_t nblk = screen_blocks(a, TU);
    const float rmax = __uint_as_float(*a.rmax_bits);
    // phase 1 only without a list: listed users come with their bound
    const int t0 = listed ? 0 : (a.t0tiles < a.ntiles ? a.t0tiles : a.ntiles);
    auto tile_of = [&](int it) { return it < t0 ? it : split + (it - t0) * a.nsplit; };

    const uint32_t magic = slot_magic(w16);
    unsigned long long pacc = 0;  // statistics: phase-2 pairs screened
    if (tid < 2 * LDS_GUARD / 16) {
        const int g = tid / (LDS_GUARD / 16), e = tid % (LDS_GUARD / 16);
        reinterpret_cast<uint4 *>(Pbase + g * bstride + TILE_ITEMS * ls)[e] =
            make_uint4(0, 0, 0, 0);
    }

    for (int64_t blk = blockIdx.x; blk < nblk; blk += gridDim.x) {
        __syncthreads();  // the previous block is done with the tile buffers
        const int64_t pos = blk * TU + ucol;
        const bool uvalid = pos < nlist;
        const int64_t ug = uvalid ? (listed ? (int64_t)a.ulist[pos] : pos) : 0;
        const int64_t nub = (nlist - blk * TU < TU) ? (nlist - blk * TU) : TU;
        int64_t ntile_p2 = 0;
        // this lane's half of its user's row, kept in registers for the whole scan
        uint4 ub[NCH];
        load_half_row<NCH>(ub, reinterpret_cast<const uint8_t *>(a.Uq), ug, uvalid, rowb, nch,
                           lane);
        // all values and bounds of a user are taken in units of its scale, a
        // power of two (the same bits, and rows of any magnitude stay in range);
        // unscaled formats: 1
        const float su = scaled_prec(PREC) && uvalid ? a.su[ug] : 1.0f, su_inv = pow2_rcp(su);
        const float nu = uvalid ? a.Nu[ug] * su_inv : 0.0f;
        const float nhu = uvalid ? a.Nhu[ug] * su_inv : 0.0f;
        const float ru = uvalid ? a.Ru[ug] * su_inv : 0.0f;
        const float e_abs = a.e_abs * su_inv;

        // error bound of this user against an item: E(u,p)
        auto ebound = [&](float n_p, float nh_p, float r_p) {
            return fmaf(ru, n_p,
                        fmaf(nhu, r_p, fmaf(a.c_err * nhu, nh_p, fmaf(a.c2 * nu, n_p, e_abs))));
        };
        // exit ratio: with N_t the largest norm of item p's tile, vh + E <=
        // K_u * N_t + 2 e_abs (R_p <= rmax N_t), so no item of a tile with N_t
        // below (L - 2 e_abs) / K_u reaches L, nor of a later one
        auto exit_ratio = [&](float L) {
            float rr = INFINITY;
            if (uvalid) {
                const float K = nu * (1.0f + a.g64 + 2.0f * a.c2) + 2.0f * ru +
                                2.0f * nhu * (rmax + a.c_err * (1.0f + rmax));
                rr = (L > 2.0f * e_abs && K > 0.0f) ? (L - 2.0f * e_abs) / K * (1.0f - 0x1p-20f)
                                                    : 0.0f;
            }
            return wave_min(rr);
        };

        float L0 = -INFINITY, rwg = INFINITY;
        if (listed) {
            L0 = uvalid ? a.Luse[ug] * su_inv : INFINITY;
            const float rr = exit_ratio(L0);
            if (lane == 0) red[w] = rr;
        }
        // the user's list for this split holds two halves of cap / 2 entries,
        // one per half-wave (each half-wave sees other item rows), so that
        // each lane appends to its own half with a register count: no
        // atomics.  The final selection reads them as 2 * nsplit lists.
        const int half = a.cap / 2, hw = lane >> 5;
        float2 *mycand = a.cand + (ug * a.nsplit + split) * a.cap + hw * half;
        int32_t *mycid = a.cand_id + (ug * a.nsplit + split) * a.cap + hw * half;
        int myc = 0;  // candidates of this lane's half, stored or not

        // (the barrier at the top of this loop: the previous block is done
        // with the tile buffers)
        tile_copy<NW>(a, tile_of(0), rowb, w16, magic, ls, Pbase, Nbase, 0, w, lane);
        dma_wait();
        __syncthreads();
        if (listed) {
            rwg = red[0];
#pragma unroll
            for (int q = 1; q < NW; ++q) rwg = fminf(rwg, red[q]);
        }
        int buf = 0;
        // phase 1: per-slot maxima of the lower bounds vh - E over the first
        // t0 tiles, then L0 = k-th largest of the user's 64 slot maxima
        if (t0 > 0) {
            float M[32];
#pragma unroll
            for (int i = 0; i < 32; ++i) M[i] = -INFINITY;
            for (int it = 0; it < t0; ++it) {
                const int t = it;
                const int tn = tile_of(it + 1);
                const bool pre = tn < a.ntiles;
                if (pre)
                    tile_copy<NW>(a, tn, rowb, w16, magic, ls, Pbase, Nbase, buf ^ 1, w, lane);
                const uint8_t *Psh = Pbase + buf * bstride;
                const float *Nsh = Nbase + buf * NSTRIDE;
                const int64_t rb = (int64_t)t * TILE_ITEMS;
                const float e_t = ebound(Nsh[0], Nsh[3 * TILE_ITEMS], Nsh[3 * TILE_ITEMS + 1]);
                const float sc = scaled_prec(PREC) ? Nsh[3 * TILE_ITEMS + 2] : 1.0f;
                f32x16 acc0 = {0}, acc1 = {0};
                MMR<PREC, NCH>::rows2(acc0, acc1, Psh, Psh + 32 * ls, ub, ls, nch, D, (a.d + 1) / 2, lane);
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const int r = mfma32_row(i, lane);
                    if (rb + r < a.m) M[i] = fmaxf(M[i], fmaf(acc0[i], sc, -e_t));
                    if (rb + r + 32 < a.m) M[16 + i] = fmaxf(M[16 + i], fmaf(acc1[i], sc, -e_t));
                }
                if (pre) dma_wait();
                __syncthreads();
                buf ^= 1;
            }
            sort32_desc(M);
            float Bv[32];
#pragma unroll
            for (int j = 0; j < 32; ++j) Bv[j] = __shfl_xor(M[31 - j], 32);
#pragma unroll
            for (int j = 0; j < 32; ++j) M[j] = fmaxf(M[j], Bv[j]);
            merge32_desc(M);
            L0 = M[0];
#pragma unroll
            for (int j = 1; j < 32; ++j)
                if (j == a.k - 1) L0 = M[j];
            const float rr = exit_ratio(L0);
            if (lane == 0) red[w] = rr;
            __syncthreads();
            rwg = red[0];
#pragma unroll
            for (int q = 1; q < NW; ++q) rwg = fminf(rwg, red[q]);
        }
        if constexpr (!LISTED) {
            // the bounds-only pass (the launch without a user list): keep L0
            // and go to the next block
            if (split == 0 && lane < 32 && uvalid) a.Luse[ug] = L0 * su;
            continue;
        }
        // phase 2 (tiles split, split + nsplit, ...): candidates vh + E >= L0
        for (int it = t0;; ++it) {
            const int t = tile_of(it);
            if (t >= a.ntiles) break;
            const float *Nsh = Nbase + buf * NSTRIDE;
            if (Nsh[0] < rwg) break;  // Cauchy-Schwarz exit (N is sorted: Nsh[0] is the largest)
            ++ntile_p2;
            const int tn = tile_of(it + 1);
            const bool pre = tn < a.ntiles;
            if (pre)
                tile_copy<NW>(a, tn, rowb, w16, magic, ls, Pbase, Nbase, buf ^ 1, w, lane);
            const uint8_t *Psh = Pbase + buf * bstride;
            const int64_t rb = (int64_t)t * TILE_ITEMS;
            // tile maxima: N is sorted (first item), Nh and R staged with the tile
            const float e_t = ebound(Nsh[0], Nsh[3 * TILE_ITEMS], Nsh[3 * TILE_ITEMS + 1]);
            const float sp_t = scaled_prec(PREC) ? Nsh[3 * TILE_ITEMS + 2] : 1.0f;
            f32x16 acc0 = {0}, acc1 = {0};
            MMR<PREC, NCH>::rows2(acc0, acc1, Psh, Psh + 32 * ls, ub, ls, nch, D, (a.d + 1) / 2, lane);
            // first on the tile bound, then per item; the tile's scale is a power
            // of two too, so multiplying by its exact reciprocal divides exactly
            // (where that overflows no product, at most 2^38, reaches it)
            const float thr = (L0 - e_t) * pow2_rcp(sp_t);
            // (a linear chain: it compiles to three-input maxima)
            float vmax = acc0[0];
#pragma unroll
            for (int i = 1; i < 16; ++i) vmax = fmaxf(vmax, acc0[i]);
#pragma unroll
            for (int i = 0; i < 16; ++i) vmax = fmaxf(vmax, acc1[i]);
            if (__ballot(vmax >= thr && uvalid) != 0ull) {
                // this lane's slots that pass the tile bound (bit i: register
                // i & 15 of block i >> 4), then each of them once
                uint32_t pend = 0u;
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    pend |= (acc0[i] >= thr) ? (1u << i) : 0u;
                    pend |= (acc1[i] >= thr) ? (1u << (16 + i)) : 0u;
                }
                if (!uvalid) pend = 0u;
                while (pend != 0u) {
                    const int i = __builtin_ctz(pend);
                    pend &= pend - 1u;
                    const int r = mfma32_row(i & 15, lane) + (i >> 4) * 32;
                    if (rb + r >= a.m) continue;  // padding rows of the last tile
                    const float v = pick32(acc0, acc1, i) * sp_t;
                    const float eb = ebound(Nsh[r], Nsh[TILE_ITEMS + r], Nsh[2 * TILE_ITEMS + r]);
                    if (v + eb >= L0) {
                        if (myc < half) {
                            mycand[myc] = make_float2(v * su, eb * su);
                            mycid[myc] = __float_as_int(Nsh[4 * TILE_ITEMS + r]);
                        }
                        ++myc;
                    }
                }
            }
            if (pre) dma_wait();
            __syncthreads();
            buf ^= 1;
        }
        if (uvalid) a.cand_cnt[(ug * a.nsplit + split) * 2 + hw] = myc;
        pacc += (unsigned long long)(ntile_p2 * TILE_ITEMS * nub);
    }
    if (a.pairs && tid == 0 && pacc)
        atomicAdd(a.pairs + (blockIdx.x & (CSTAT_SLOTS - 1)), pacc);
}

// The passes with a user list (phase 2 alone) for BF16 and the f8f6f4
// formats, with two blocks of 32 users per wave: each item chunk read from
// LDS feeds four products (two item blocks x two user blocks), half the LDS
// reads per product of k_thresh_screen.  8 waves of 64 users (two per SIMD:
// both users' half rows stay in registers; split FP32 rows fit without
// spills up to 10 chunks, d = 80).  The band test, the candidate
// lists and the exit are k_thresh_screen's, per user block.
constexpr int SCR2_NW = 8;
__host__ __device__ constexpr bool screen_u2(int prec, int nch) {
    return prec == PREC_SPLIT ? nch <= 10 : prec != PREC_FP32 && nch <= 16;
}
template <int PREC, int NCH>
__global__ __launch_bounds__(64 * SCR2_NW) __attribute__((amdgpu_waves_per_eu(2)))
void k_thresh_screen_u2(ThreshArgs a) {
    constexpr int NW = SCR2_NW, TU = 64 * NW;
    extern __shared__ __align__(16) uint8_t smem8[];
    const int D = a.D, ls = lds_row_bytes(PREC, D), rowb = D * elem_bytes(PREC);
    const int nch = rowb / 32;
    const int bstride = TILE_ITEMS * ls + LDS_GUARD;
    uint8_t *Pbase = smem8;
    float *Nbase = reinterpret_cast<float *>(Pbase + 2 * bstride);
    float *red = reinterpret_cast<float *>(Nbase + 2 * NSTRIDE);

    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int split = blockIdx.y;
    const int w16 = rowb / 16;
    const int64_t nlist = (int64_t)*a.ulist_cnt;
    const int64_t nblk = (nlist + TU - 1) / TU;
    const float rmax = __uint_as_float(*a.rmax_bits);
    auto tile_of = [&](int it) { return split + it * a.nsplit; };

    const uint32_t magic = slot_magic(w16);
    unsigned long long pacc = 0;  // statistics: pairs screened
    if (tid < 2 * LDS_GUARD / 16) {
        const int g = tid / (LDS_GUARD / 16), e = tid % (LDS_GUARD / 16);
        reinterpret_cast<uint4 *>(Pbase + g * bstride + TILE_ITEMS * ls)[e] =
            make_uint4(0, 0, 0, 0);
    }
    const int half = a.cap / 2, hw = lane >> 5;

    for (int64_t blk = blockIdx.x; blk < nblk; blk += gridDim.x) {
        __syncthreads();  // the previous block is done with the tile buffers
        const int64_t nub = (nlist - blk * TU < TU) ? (nlist - blk * TU) : TU;
        int64_t ntile_p2 = 0;
        // user block h of this wave: users w * 64 + 32 h + (lane & 31)
        bool uvalid[2];
        int64_t ug[2];
        uint4 ub0[NCH], ub1[NCH];
        // (in units of the user's scale, as in k_thresh_screen)
        float nu[2], nhu[2], ru[2], su[2], e_abs[2], L0[2];
        float2 *mycand[2];
        int32_t *mycid[2];
        int myc[2] = {0, 0};
        float rr = INFINITY;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int64_t pos = blk * TU + w * 64 + 32 * h + (lane & 31);
            uvalid[h] = pos < nlist;
            ug[h] = uvalid[h] ? (int64_t)a.ulist[pos] : 0;
            su[h] = scaled_prec(PREC) && uvalid[h] ? a.su[ug[h]] : 1.0f;
            const float su_inv = pow2_rcp(su[h]);
            nu[h] = uvalid[h] ? a.Nu[ug[h]] * su_inv : 0.0f;
            nhu[h] = uvalid[h] ? a.Nhu[ug[h]] * su_inv : 0.0f;
            ru[h] = uvalid[h] ? a.Ru[ug[h]] * su_inv : 0.0f;
            e_abs[h] = a.e_abs * su_inv;
            L0[h] = uvalid[h] ? a.Luse[ug[h]] * su_inv : INFINITY;
            mycand[h] = a.cand + (ug[h] * a.nsplit + split) * a.cap + hw * half;
            mycid[h] = a.cand_id + (ug[h] * a.nsplit + split) * a.cap + hw * half;
            // exit ratio as in k_thresh_screen
            if (uvalid[h]) {
                const float K = nu[h] * (1.0f + a.g64 + 2.0f * a.c2) + 2.0f * ru[h] +
                                2.0f * nhu[h] * (rmax + a.c_err * (1.0f + rmax));
                const float r = (L0[h] > 2.0f * e_abs[h] && K > 0.0f)
                                    ? (L0[h] - 2.0f * e_abs[h]) / K * (1.0f - 0x1p-20f)
                                    : 0.0f;
                rr = fminf(rr, r);
            }
        }
        load_half_row<NCH>(ub0, reinterpret_cast<const uint8_t *>(a.Uq), ug[0], uvalid[0], rowb,
                           nch, lane);
        load_half_row<NCH>(ub1, reinterpret_cast<const uint8_t *>(a.Uq), ug[1], uvalid[1], rowb,
                           nch, lane);
        rr = wave_min(rr);
        if (lane == 0) red[w] = rr;
        auto ebound = [&](int h, float n_p, float nh_p, float r_p) {
            return fmaf(ru[h], n_p, fmaf(nhu[h], r_p,
                                         fmaf(a.c_err * nhu[h], nh_p, fmaf(a.c2 * nu[h], n_p, e_abs[h]))));
        };
        tile_copy<NW>(a, tile_of(0), rowb, w16, magic, ls, Pbase, Nbase, 0, w, lane);
        dma_wait();
        __syncthreads();
        float rwg = red[0];
#pragma unroll
        for (int q = 1; q < NW; ++q) rwg = fminf(rwg, red[q]);
        int buf = 0;
        for (int it = 0;; ++it) {
            const int t = tile_of(it);
            if (t >= a.ntiles) break;
            const float *Nsh = Nbase + buf * NSTRIDE;
            if (Nsh[0] < rwg) break;  // Cauchy-Schwarz exit (N is sorted: Nsh[0] is the largest)
            ++ntile_p2;
            const int tn = tile_of(it + 1);
            const bool pre = tn < a.ntiles;
            if (pre)
                tile_copy<NW>(a, tn, rowb, w16, magic, ls, Pbase, Nbase, buf ^ 1, w, lane);
            const uint8_t *Psh = Pbase + buf * bstride;
            const int64_t rb = (int64_t)t * TILE_ITEMS;
            const float sp_t = scaled_prec(PREC) ? Nsh[3 * TILE_ITEMS + 2] : 1.0f;
            f32x16 acc[2][2];
#pragma unroll
            for (int h = 0; h < 2; ++h) acc[h][0] = acc[h][1] = f32x16{0};
            MMR<PREC, NCH>::rows4(acc, Psh, Psh + 32 * ls, ub0, ub1, ls, D, lane);
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const float e_t = ebound(h, Nsh[0], Nsh[3 * TILE_ITEMS], Nsh[3 * TILE_ITEMS + 1]);
                const float thr = (L0[h] - e_t) * pow2_rcp(sp_t);
                float vmax = acc[h][0][0];
#pragma unroll
                for (int i = 1; i < 16; ++i) vmax = fmaxf(vmax, acc[h][0][i]);
#pragma unroll
                for (int i = 0; i < 16; ++i) vmax = fmaxf(vmax, acc[h][1][i]);
                if (__ballot(vmax >= thr && uvalid[h]) != 0ull) {
                    uint32_t pend = 0u;
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        pend |= (acc[h][0][i] >= thr) ? (1u << i) : 0u;
                        pend |= (acc[h][1][i] >= thr) ? (1u << (16 + i)) : 0u;
                    }
                    if (!uvalid[h]) pend = 0u;
                    while (pend != 0u) {
                        const int i = __builtin_ctz(pend);
                        pend &= pend - 1u;
                        const int r = mfma32_row(i & 15, lane) + (i >> 4) * 32;
                        if (rb + r >= a.m) continue;  // padding rows of the last tile
                        const float v = pick32(acc[h][0], acc[h][1], i) * sp_t;
                        const float eb =
                            ebound(h, Nsh[r], Nsh[TILE_ITEMS + r], Nsh[2 * TILE_ITEMS + r]);
                        if (v + eb >= L0[h]) {
                            if (myc[h] < half) {
                                mycand[h][myc[h]] = make_float2(v * su[h], eb * su[h]);
                                mycid[h][myc[h]] = __float_as_int(Nsh[4 * TILE_ITEMS + r]);
                            }
                            ++myc[h];
                        }
                    }
                }
            }
            if (pre) dma_wait();
            __syncthreads();
            buf ^= 1;
        }
#pragma unroll
        for (int h = 0; h < 2; ++h)
            if (uvalid[h]) a.cand_cnt[(ug[h] * a.nsplit + split) * 2 + hw] = myc[h];
        pacc += (unsigned long long)(ntile_p2 * TILE_ITEMS * nub);
    }
    if (a.pairs && tid == 0 && pacc)
        atomicAdd(a.pairs + (blockIdx.x & (CSTAT_SLOTS - 1)), pacc);
}

// ------------------------------------------------------------------ final
// Wave-level bitonic sort of (value, id) pairs in LDS in the order (value
// desc, id asc); the slots from n up to the next power of two are filled
// first.
__device__ void wave_sort_pairs(double *v, int *id, int n, int lane) {
    int P2 = 1;
    while (P2 < n) P2 <<= 1;
    for (int i = n + lane; i < P2; i += 64) {
        v[i] = -INFINITY;
        id[i] = 0x7fffffff;
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_wave_barrier();
    for (int kk = 2; kk <= P2; kk <<= 1)
        for (int j = kk >> 1; j > 0; j >>= 1) {
            for (int i = lane; i < P2; i += 64) {
                const int l = i ^ j;
                if (l > i) {
                    const double x = v[i], y = v[l];
                    const int xi = id[i], yi = id[l];
                    const bool y_first = (y > x) || (y == x && yi < xi);
                    const bool desc = (i & kk) == 0;
                    if (y_first == desc) {
                        v[i] = y; v[l] = x;
                        id[i] = yi; id[l] = xi;
                    }
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
            __builtin_amdgcn_wave_barrier();
        }
}


constexpr int FIN_WAVES = 4;
constexpr int FIN_WPE = 4;  // waves per SIMD of the final selection
constexpr int FIN_ENTRY_BYTES = 12;  // LDS bytes per list entry of the final selection
size_t final_entry_bytes() { return FIN_ENTRY_BYTES; }
// recomputations per user handed from the selection to k_thresh_exact; more, up
// to EXACT_WIDE, go to k_thresh_exact_wide
constexpr int EXACT_SLOTS = 8;
constexpr int EXACT_WIDE = 2048;
constexpr int EXACT_REGS = 1024;  // values ranked in registers

// Orders this wave's LDS accesses (every list of the final selection is
// private to one wave, so no workgroup barrier is needed).
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Wave-wide maximum and sum by DPP steps (no LDS traffic): quad_perm
// [1,0,3,2] and [2,3,0,1] combine the lanes of each quad, row_half_mirror
// and row_mirror the quads of each row of 16, row_bcast:15 (rows 1, 3) and
// row_bcast:31 (rows 2, 3) the rows; lane 63 then holds the result, read
// back as a wave-uniform value.  Lanes left out of a step keep `old`, the
// operation's identity.
template <int CTRL, int ROWS>
__device__ __forceinline__ int dpp_from(int identity, int v) {
    return __builtin_amdgcn_update_dpp(identity, v, CTRL, ROWS, 0xf, false);
}
__device__ __forceinline__ int dpp_wave_sum(int x) {
    x += dpp_from<0xB1, 0xf>(0, x);
    x += dpp_from<0x4E, 0xf>(0, x);
    x += dpp_from<0x141, 0xf>(0, x);
    x += dpp_from<0x140, 0xf>(0, x);
    x += dpp_from<0x142, 0xa>(0, x);
    x += dpp_from<0x143, 0xc>(0, x);
    return __builtin_amdgcn_readlane(x, 63);
}

__device__ __forceinline__ uint32_t dpp_wave_max_u32(uint32_t x) {
    x = max(x, (uint32_t)dpp_from<0xB1, 0xf>(0, (int)x));
    x = max(x, (uint32_t)dpp_from<0x4E, 0xf>(0, (int)x));
    x = max(x, (uint32_t)dpp_from<0x141, 0xf>(0, (int)x));
    x = max(x, (uint32_t)dpp_from<0x140, 0xf>(0, (int)x));
    x = max(x, (uint32_t)dpp_from<0x142, 0xa>(0, (int)x));
    x = max(x, (uint32_t)dpp_from<0x143, 0xc>(0, (int)x));
    return (uint32_t)__builtin_amdgcn_readlane((int)x, 63);
}

// The k-th largest of the wave's keys (float_key; 0, below every float's, for
// a slot that holds none), at least k of them: the largest key that k of them
// reach, bit by bit from the first bit in which the smallest and the largest
// differ, each bit decided by the number of keys that reach it (a compare and
// a scalar population count per register).  Once exactly k keys are left they
// are the k largest, and their smallest is the answer.
template <int J>
__device__ __forceinline__ uint32_t wave_kth_key(const uint32_t (&r)[J], int k) {
    uint32_t mx = 0u, mn = 0u;  // mn: of the complements
#pragma unroll
    for (int j = 0; j < J; ++j) {
        mx = max(mx, r[j]);
        mn = max(mn, r[j] != 0u ? ~r[j] : 0u);
    }
    mx = dpp_wave_max_u32(mx);
    mn = ~dpp_wave_max_u32(mn);
    if (mx == mn) return mx;
    int b = 31 - __builtin_clz(mx ^ mn);
    uint32_t t = b == 31 ? 0u : mn & ~((2u << b) - 1u);  // the common prefix
    for (; b >= 0; --b) {
        const uint32_t c = t | (1u << b);
        int cnt = 0;
#pragma unroll
        for (int j = 0; j < J; ++j) cnt += __popcll(__ballot(r[j] >= c));
        if (cnt >= k) t = c;
        if (cnt == k) {
            uint32_t m = 0u;
#pragma unroll
            for (int j = 0; j < J; ++j) m = max(m, r[j] >= c ? ~r[j] : 0u);
            return ~dpp_wave_max_u32(m);
        }
    }
    return t;
}

// The k-th largest of x and of y (keys as above; n >= k of each, in the first n
// lanes): the smallest key with fewer than k larger ones, every lane counting
// the larger ones of its own two keys.  Three instructions per key and list
// that do not wait for each other, where wave_kth_key's chain of compare,
// count and branch takes some 25 steps (500k users, lists of 27: 0.60 to 0.44
// ms for k_thresh_select).
__device__ __forceinline__ void wave_kth_pair(uint32_t x, uint32_t y, int n, int k, uint32_t &kx,
                                              uint32_t &ky) {
    int gx = 0, gy = 0;
#pragma unroll 4
    for (int q = 0; q < n; ++q) {
        gx += (uint32_t)__builtin_amdgcn_readlane((int)x, q) > x ? 1 : 0;
        gy += (uint32_t)__builtin_amdgcn_readlane((int)y, q) > y ? 1 : 0;
    }
    kx = ~dpp_wave_max_u32(x != 0u && gx < k ? ~x : 0u);
    ky = ~dpp_wave_max_u32(y != 0u && gy < k ? ~y : 0u);
}

// The k-th largest of the list x[0..n) in LDS, counting repetitions (-inf
// when n < k); lists past 1024 values are read again for every bit.
template <int J>
__device__ __forceinline__ float wave_kth_regs(const float *x, int n, int k, int lane) {
    uint32_t r[J];
#pragma unroll
    for (int j = 0; j < J; ++j) r[j] = lane + 64 * j < n ? float_key(x[lane + 64 * j]) : 0u;
    return key_float(wave_kth_key(r, k));
}
__device__ float wave_kth_largest(const float *x, int n, int k, int lane) {
    if (n < k) return -INFINITY;
    if (n <= 64) return wave_kth_regs<1>(x, n, k, lane);
    if (n <= 128) return wave_kth_regs<2>(x, n, k, lane);
    if (n <= 256) return wave_kth_regs<4>(x, n, k, lane);
    if (n <= 512) return wave_kth_regs<8>(x, n, k, lane);
    if (n <= 1024) return wave_kth_regs<16>(x, n, k, lane);
    uint32_t t = 0u;
    for (int b = 31; b >= 0; --b) {
        const uint32_t c = t | (1u << b);
        int cnt = 0;
        for (int e = lane; e < n; e += 64) cnt += float_key(x[e]) >= c ? 1 : 0;
        if (dpp_wave_sum(cnt) >= k) t = c;
    }
    return key_float(t);
}

// The selection where a user's lists hold at most SEL_MAX entries
// (k_thresh_final takes the others): as k_thresh_final, but with the joined
// list in registers (J entries per lane) from its load to the ids left for
// the recomputation, so that no LDS limits the waves in flight.  Latency and
// the selection's instructions bound it: 500k users, e4m3 lists of 241
// entries 1.3 ms (1.6 with four workgroups to a CU; lists of 429 2.5 ms then,
// and 9.9 ms in LDS by rounds of the next largest); BF16 lists of 27 entries
// 0.44 ms, 2M users with lists of 11 1.17 ms (0.72 and 2.0 ms), of which reading
// the counts two users and the entries one user ahead is 0.03 and 0.2 ms.
constexpr int SEL_MAX = 2048;
// lists up to SEL_SHORT leave registers for four waves per SIMD (118), up to
// SEL_MID for three (166 of 168), longer ones for two; a launch is one round of
// the workgroups that are resident then (with four to a CU throughout, three
// resident and a partial second round: e4m3, k = 20, 300k users 1.14 ms for
// 0.92; k = 24 1.29 for 1.05, and 1.39 with two waves)
constexpr int SEL_SHORT = 1024, SEL_MID = 1536;
struct SelOut {
    float Lstar;      // k-th largest lower bound of the stored entries (-inf: fewer than k)
    int nrec, ns;     // entries left to recompute, survivors
};
// entry g of the user's joined list (pre: the lists' inclusive prefixes, one
// per lane; split = number of them that are <= g)
__device__ __forceinline__ void joined_entry(const ThreshArgs &a, int64_t u, int pre, int stored,
                                             int g, float2 &cv, int &ci) {
    int sp = 0, before = 0;
    for (int q = 0; q < a.nsplit; ++q) {
        const int pq = __builtin_amdgcn_readlane(pre, q);
        if (pq <= g) {
            sp = q + 1;
            before = pq;
        }
    }
    cv = make_float2(0.0f, 0.0f);
    ci = 0;
    if (g < stored) {
        const int64_t e = (u * a.nsplit + sp) * a.cap + (g - before);
        cv = a.cand[e];
        ci = a.cand_id[e];
    }
}
// (J = 1: the entry is e0, id0)
template <int J>
__device__ __forceinline__ SelOut select_regs(const ThreshArgs &a, int64_t u, int pre, int stored,
                                              bool over, float2 e0, int id0, int lane) {
    uint32_t lo[J], hi[J];  // keys of the bounds vh -/+ E, 0 past the end
    int ci[J];
#pragma unroll
    for (int t = 0; t < J; ++t) {
        const int g = 64 * t + lane;
        float2 cv = e0;
        ci[t] = id0;
        if (J > 1) joined_entry(a, u, pre, stored, g, cv, ci[t]);
        lo[t] = g < stored ? float_key(cv.x - cv.y) : 0u;
        hi[t] = g < stored ? float_key(cv.x + cv.y) : 0u;
    }
    SelOut o{-INFINITY, 0, 0};
    // (the k-th largest upper bound is the same with and without the entries
    // below L*: at least k reach it)
    uint32_t L = 0u, Hk = ~0u;
    const bool pair = J == 1 && !a.topk;  // (for L* alone the chain is the shorter: 0.15, 0.19 ms)
    if (stored >= a.k) {
        if (pair) wave_kth_pair(lo[0], hi[0], stored, a.k, L, Hk);
        else L = wave_kth_key(lo, a.k);
    }
    if (stored >= a.k) o.Lstar = key_float(L);
    if (over) return o;
    // survivors: upper bound reaches L*; left to recompute: those whose lower
    // bound is at most H_k, the k-th largest upper bound (all of them where
    // the whole of S_k is asked for)
#pragma unroll
    for (int t = 0; t < J; ++t) {
        if (hi[t] < L) hi[t] = 0u;
        o.ns += __popcll(__ballot(hi[t] != 0u));
    }
    if (J > 1 && !a.topk) Hk = wave_kth_key(hi, a.k);
    const int64_t c0 = u * a.nsplit * (int64_t)a.cap;
#pragma unroll
    for (int t = 0; t < J; ++t) {
        const bool unc = hi[t] != 0u && lo[t] <= Hk;
        const uint64_t bal = __ballot(unc);
        const int q = o.nrec + __popcll(bal & ((lane == 0) ? 0ull : (~0ull >> (64 - lane))));
        // (every entry of the list is in a register by now)
        if (unc) a.cand_id[c0 + q] = ci[t];
        o.nrec += __popcll(bal);
    }
    return o;
}

constexpr int sel_waves(int max) { return max <= SEL_SHORT ? 4 : max <= SEL_MID ? 3 : 2; }
template <int MAX>  // longest list
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(sel_waves(MAX))))
void k_thresh_select(ThreshArgs a) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nw = blockDim.x >> 6;
    const int64_t nlist = (int64_t)*a.ulist_cnt;
    unsigned long long *cs = a.cstats ? a.cstats + (blockIdx.x & (CSTAT_SLOTS - 1)) * 4 : nullptr;
    unsigned long long st_cand = 0, st_rec = 0;
    const int64_t step = (int64_t)gridDim.x * nw;
    int64_t pos = (int64_t)blockIdx.x * nw + w;
    // the split counts of a user, one per lane (at most 16), are read two users
    // ahead, and the entries of a list of up to 64 one user ahead
    auto user_at = [&](int64_t p) { return p < nlist ? (int64_t)a.ulist[p] : 0; };
    auto counts_of = [&](int64_t p, int64_t x) {
        return (p < nlist && lane < a.nsplit) ? a.cand_cnt[x * a.nsplit + lane] : 0;
    };
    // inclusive prefix of the stored counts (in the first row of 16 lanes)
    auto prefix_of = [&](int c) {
        int p = c < a.cap ? c : a.cap;
        p += dpp_from<0x111, 0xf>(0, p);
        p += dpp_from<0x112, 0xf>(0, p);
        p += dpp_from<0x114, 0xf>(0, p);
        p += dpp_from<0x118, 0xf>(0, p);
        return p;
    };
    int64_t u = user_at(pos), un = user_at(pos + step);
    int cl = counts_of(pos, u), cn = counts_of(pos + step, un);
    int pre = prefix_of(cl), stored = __builtin_amdgcn_readlane(pre, 15);
    float2 cv = make_float2(0.0f, 0.0f);
    int id = 0;
    if (stored <= 64) joined_entry(a, u, pre, stored, lane, cv, id);
    for (; pos < nlist; pos += step) {
        const int64_t u2 = user_at(pos + 2 * step);
        const int c2 = counts_of(pos + 2 * step, u2);
        const int pren = prefix_of(cn), storedn = __builtin_amdgcn_readlane(pren, 15);
        float2 cvn = make_float2(0.0f, 0.0f);
        int idn = 0;
        if (storedn <= 64) joined_entry(a, un, pren, storedn, lane, cvn, idn);
        const bool over = __ballot(cl > a.cap) != 0ull;
        SelOut o;
        if (stored <= 64) o = select_regs<1>(a, u, pre, stored, over, cv, id, lane);
        else if (stored <= 128) o = select_regs<2>(a, u, pre, stored, over, cv, id, lane);
        else if (stored <= 256) o = select_regs<4>(a, u, pre, stored, over, cv, id, lane);
        else if (stored <= 512) o = select_regs<8>(a, u, pre, stored, over, cv, id, lane);
        else if (MAX == SEL_SHORT || stored <= SEL_SHORT)
            o = select_regs<SEL_SHORT / 64>(a, u, pre, stored, over, cv, id, lane);
        else o = select_regs<MAX / 64>(a, u, pre, stored, over, cv, id, lane);
        if (over) {
            // screened again from a tighter bound, or the exact fallback
            if (lane == 0) {
                const float Lprev = a.Luse[u];
                const float Lnew = fmaxf(o.Lstar, Lprev);
                if (a.rlist && Lnew > Lprev) {
                    a.Luse[u] = Lnew;
                    a.rlist[atomicAdd(a.rcnt, 1)] = (int)u;
                    if (cs) atomicAdd(cs + 3, 1ull);
                } else {
                    a.flist[atomicAdd(a.fcnt, 1)] = (int)u;
                    if (cs) atomicAdd(cs + 2, 1ull);
                }
            }
        } else {
            st_cand += (unsigned long long)stored;  // (no list overflowed)
            st_rec += (unsigned long long)o.nrec;
        }
        // rank of tau among the values to recompute, and their count (-1: none)
        if (lane == 0)
            a.cand_cnt[u * a.nsplit] = over ? -1 : (a.k - 1 - (o.ns - o.nrec)) | (o.nrec << 8);
        u = un;
        cl = cn;
        pre = pren;
        stored = storedn;
        cv = cvn;
        id = idn;
        un = u2;
        cn = c2;
    }
    if (cs && lane == 0) {
        if (st_cand) atomicAdd(cs, st_cand);
        if (st_rec) atomicAdd(cs + 1, st_rec);
    }
}

// One wave per user.  The lists of the user's splits are gathered into
// LDS with lower and upper bounds vh -/+ E; L* = k-th largest lower bound.
// A user whose lists overflowed is not resolved here: the k-th largest lower
// bound among its stored candidates (distinct items, so at most tau_u) is a
// tighter starting bound for another screening pass, or, when it does not
// improve on the bound used, the user goes to the exact fallback.
// capT: longest candidate list taken; capP: array stride, capT rounded up
// to a power of two so that the bitonic sorts can pad in place.
// Four waves per SIMD: the FP64 recomputations load 16 values per row at a
// time (latency), which needs more than the registers of six.
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(FIN_WPE)))
void k_thresh_final(ThreshArgs a, int capT, int capP) {
    extern __shared__ float smem[];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int nw = blockDim.x >> 6;  // waves per block (one user each)
    // per-wave LDS (FIN_ENTRY_BYTES per entry): lo, hi (float), cidx (int),
    // the survivors and then the values to recompute compacted in place; the
    // FP64 values v64 take the place of lo and hi once those are no longer
    // read
    uint8_t *base = reinterpret_cast<uint8_t *>(smem) + (size_t)w * capP * FIN_ENTRY_BYTES;
    float *lo = reinterpret_cast<float *>(base);
    float *hi = lo + capP;
    double *v64 = reinterpret_cast<double *>(base);
    int *cidx = reinterpret_cast<int *>(hi + capP);
    __shared__ float Lstar[FIN_WAVES];
    __shared__ int nsurv[FIN_WAVES];
    const int64_t nlist = (int64_t)*a.ulist_cnt;
    unsigned long long *cs = a.cstats ? a.cstats + (blockIdx.x & (CSTAT_SLOTS - 1)) * 4 : nullptr;
    // statistics of this wave's users (candidates, recomputed), added to
    // the counters once at the end
    unsigned long long st_cand = 0, st_rec = 0;

    for (int64_t b0 = (int64_t)blockIdx.x * nw; b0 < nlist; b0 += (int64_t)gridDim.x * nw) {
        const int64_t pos = b0 + w;
        const bool valid = pos < nlist;
        const int64_t u = valid ? (int64_t)a.ulist[pos] : 0;
        // the split counts, one per lane (nsplit <= 64), and their sums;
        // stored entries are laid out split after split
        int cl = 0;
        if (valid && lane < a.nsplit) cl = a.cand_cnt[u * a.nsplit + lane];
        bool over = __ballot(cl > a.cap) != 0ull;
        const int sl = cl < a.cap ? cl : a.cap;
        int pre = sl;  // inclusive prefix of the stored counts
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int y = __shfl_up(pre, o);
            if (lane >= o) pre += y;
        }
        const int stored = __builtin_amdgcn_readlane(pre, 63);
        int total = 0;  // statistics: candidates found, stored or not
        if (cs) {
            int t = cl;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) t += __shfl_xor(t, o);
            total = __builtin_amdgcn_readlane(t, 0);
        }
        if (stored > capT) over = true;  // cannot happen: nsplit * cap <= capT
        wave_sync();  // this wave's previous user is done with its LDS lists
        if (lane == 0) Lstar[w] = -INFINITY;
        if (valid && stored <= capT) {
            // entry g of the joined list (64 at a time, from every split
            // at once): split s = number of inclusive prefixes <= g, entry
            // g - (prefix before s); FIN_GU rounds of loads are issued before
            // their entries are stored, so that their latencies overlap
            constexpr int FIN_GU = 4;
            for (int g0 = 0; g0 < stored; g0 += 64 * FIN_GU) {
                float2 cv[FIN_GU];  // (screened value, its bound E)
                int ci[FIN_GU];
#pragma unroll
                for (int t = 0; t < FIN_GU; ++t) {
                    const int g = g0 + 64 * t + lane;
                    int sp = 0, before = 0;
                    for (int q = 0; q < a.nsplit; ++q) {
                        const int pq = __builtin_amdgcn_readlane(pre, q);
                        if (pq <= g) {
                            sp = q + 1;
                            before = pq;
                        }
                    }
                    cv[t] = make_float2(0.0f, 0.0f);
                    ci[t] = 0;
                    if (g < stored) {
                        const int64_t e = (u * a.nsplit + sp) * a.cap + (g - before);
                        cv[t] = a.cand[e];
                        ci[t] = a.cand_id[e];
                    }
                }
#pragma unroll
                for (int t = 0; t < FIN_GU; ++t) {
                    const int g = g0 + 64 * t + lane;
                    if (g < stored) {
                        lo[g] = cv[t].x - cv[t].y;
                        hi[g] = cv[t].x + cv[t].y;
                        cidx[g] = ci[t];
                    }
                }
            }
        }
        wave_sync();
        // L* = k-th largest lower bound: by ranks for short lists, else bit by
        // bit (wave_kth_largest; the list stays in place, paired with the upper
        // bounds and ids)
        if (valid && stored <= capT) {
            if (stored <= 128) {
                for (int e = lane; e < stored; e += 64) {
                    const float x = lo[e];
                    int rank = 0;
                    for (int f = 0; f < stored; ++f) {
                        const float y = lo[f];
                        rank += (y > x) || (y == x && f < e);
                    }
                    if (rank == a.k - 1) Lstar[w] = x;
                }
            } else {
                const float Ls = wave_kth_largest(lo, stored, a.k, lane);
                if (lane == 0) Lstar[w] = Ls;
            }
        }
        wave_sync();
        if (valid && over) {
            if (lane == 0) {
                const float Lprev = a.Luse[u];
                const float Lnew = stored >= a.k ? fmaxf(Lstar[w], Lprev) : Lprev;
                if (a.rlist && Lnew > Lprev) {
                    a.Luse[u] = Lnew;
                    a.rlist[atomicAdd(a.rcnt, 1)] = (int)u;
                    if (cs) atomicAdd(cs + 3, 1ull);
                } else {
                    a.flist[atomicAdd(a.fcnt, 1)] = (int)u;
                    if (cs) atomicAdd(cs + 2, 1ull);
                }
            }
        }
        const bool work = valid && !over;
        if (work) st_cand += (unsigned long long)total;
        // survivors: upper bound reaches L*; their caller ids and bounds
        // compacted in place (a survivor's slot is at most its index, and each
        // round of 64 reads its entries before it writes)
        if (work) {
            const float Ls = Lstar[w];
            int cntw = 0;
            // (no list overflowed: every candidate is stored)
            for (int e0 = 0; e0 < stored; e0 += 64) {
                const int e = e0 + lane;
                float l = 0.0f, h = 0.0f;
                int c = 0;
                if (e < stored) {
                    l = lo[e];
                    h = hi[e];
                    c = cidx[e];
                }
                const bool keep = e < stored && h >= Ls;
                const uint64_t bal = __ballot(keep);
                const int p = cntw + __popcll(bal & ((lane == 0) ? 0ull : (~0ull >> (64 - lane))));
                __builtin_amdgcn_wave_barrier();
                if (keep) {
                    cidx[p] = c;
                    lo[p] = l;
                    hi[p] = h;
                }
                cntw += __popcll(bal);
            }
            if (lane == 0) nsurv[w] = cntw;
        }
        wave_sync();
        // When only tau is asked for, a survivor whose lower bound exceeds the
        // upper bounds of all but at most k - 2 others ranks above the k-th
        // item; with A such survivors, tau is the (k - A)-th of the others, and
        // only those are recomputed.  A survivor p is such another one when
        // at least k upper bounds (its own included) reach lo[p], that is
        // when lo[p] <= H_k, the k-th largest upper bound of the survivors
        // (counted directly for short lists, where that is cheaper).
        const bool band = a.topk == nullptr;
        int *rid = cidx;
        if (work) {
            const int ns = nsurv[w];
            int nrec = ns;
            if (band) {
                const bool direct = ns <= 128;
                const float Hk = direct ? 0.0f : wave_kth_largest(hi, ns, a.k, lane);
                int cntb = 0;
                for (int p0 = 0; p0 < ns; p0 += 64) {
                    const int p = p0 + lane;
                    bool unc = false;
                    int id = 0;
                    if (p < ns) {
                        const float x = lo[p];
                        if (direct) {
                            int c = 0;
                            for (int q = 0; q < ns; ++q) c += hi[q] >= x;
                            unc = c >= a.k;
                        } else {
                            unc = x <= Hk;
                        }
                        id = cidx[p];
                    }
                    const uint64_t bal = __ballot(unc);
                    const int q = cntb + __popcll(bal & ((lane == 0) ? 0ull : (~0ull >> (64 - lane))));
                    if (unc) cidx[q] = id;
                    cntb += __popcll(bal);
                }
                nrec = cntb;
            }
            if (lane == 0) nsurv[w] = nrec | ((ns - nrec) << 16);
            st_rec += (unsigned long long)nrec;
        }
        wave_sync();
        // Only tau asked for: the values to recompute are left to
        // k_thresh_exact (at most EXACT_SLOTS, several users per wave) or
        // k_thresh_exact_wide (up to EXACT_WIDE, a wave per user), which hold
        // no lists in LDS and so keep many more row gathers in flight than
        // this kernel.  The ids go to this user's candidate slots (read
        // above), the target rank and the count to its first count slot; -1
        // there for every other user of the list.
        const int nrec_w = nsurv[w] & 0xffff;
        const bool defer = work && band && nrec_w <= EXACT_WIDE;
        if (valid) {
            if (defer) {
                const int64_t c0 = u * a.nsplit * (int64_t)a.cap;
                for (int q = lane; q < nrec_w; q += 64) a.cand_id[c0 + q] = rid[q];
                if (lane == 0)
                    a.cand_cnt[u * a.nsplit] = (a.k - 1 - (nsurv[w] >> 16)) | (nrec_w << 8);
            } else if (lane == 0) {
                a.cand_cnt[u * a.nsplit] = -1;
            }
        }
        wave_sync();  // (v64 takes the place of lo and hi)
        if (work && !defer) {
            const float *urow = a.U + u * a.d;
            for (int q = lane; q < nrec_w; q += 64)
                v64[q] = ip64<16>(urow, a.P + (int64_t)rid[q] * a.d, a.d);
        }
        wave_sync();
        if (work && !defer) {
            const int nrec = nsurv[w] & 0xffff, nabove = nsurv[w] >> 16;
            const int tgt = a.k - 1 - nabove;  // rank of tau among the recomputed
            if (nrec <= 128) {
                for (int q = lane; q < nrec; q += 64) {
                    const double x = v64[q];
                    const int c = rid[q];
                    int rank = 0;
                    for (int f = 0; f < nrec; ++f) {
                        const double y = v64[f];
                        rank += (y > x) || (y == x && rid[f] < c);
                    }
                    if (rank == tgt) {
                        a.tau[u] = x;
                        a.tau_id[u] = c;
                    }
                    if (a.topk && rank < a.k) a.topk[u * a.k + rank] = c;
                    if (a.topv && rank < a.k) a.topv[u * a.k + rank] = x;
                }
            } else {
                wave_sort_pairs(v64, rid, nrec, lane);
                if (lane == 0) {
                    a.tau[u] = v64[tgt];
                    a.tau_id[u] = rid[tgt];
                }
                if (a.topk)
                    for (int r = lane; r < a.k; r += 64) a.topk[u * a.k + r] = rid[r];
                if (a.topv)
                    for (int r = lane; r < a.k; r += 64) a.topv[u * a.k + r] = v64[r];
            }
        }
    }
    if (cs && lane == 0) {
        if (st_cand) atomicAdd(cs, st_cand);
        if (st_rec) atomicAdd(cs + 1, st_rec);
    }
}

// Rows for exact products.  A lane's value is a sequential FP64 sum over its
// own item row, but 64 lanes that each read their own row take 64 cache lines
// per load, one a cycle: that, and not the memory behind it, bounded the
// recomputations (L2 hit rate 0.98).  Here the wave copies a block of 32
// values of all 64 rows into LDS with whole-line loads (8 lanes a row, 8 rows
// a load; 32 lanes a row where rows are not whole aligned 16-byte vectors) and
// each lane reads its row from there (the first nrows lanes' rows).  The rows are permuted within their 128
// bytes so that the lanes' reads fall on distinct banks: 16-byte vector c of
// row r lies at c ^ (r / 2 mod 8), single values e at e ^ (r mod 32).
constexpr int XB = 32;             // values per block
constexpr int XB_FLOATS = 64 * XB;  // LDS floats of a staged block
template <bool VEC>
__device__ __forceinline__ void stage_rows(const float *X, int row, int nrows, int d, int e0,
                                           float *dst, int lane) {
    if constexpr (VEC) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            if (8 * i >= nrows) break;
            const int r = 8 * i + (lane >> 3), c = (lane & 7) ^ ((r >> 1) & 7);
            const int64_t src = __shfl(row, r);
            const int e = e0 + 4 * c;  // (past the row: its last vector again)
            dma16(X + src * d + (e < d ? e : d - 4), dst + 256 * i);
        }
    } else {
#pragma unroll 8
        for (int i = 0; i < 32; ++i) {
            if (2 * i >= nrows) break;
            const int r = 2 * i + (lane >> 5), c = (lane & 31) ^ (r & 31);
            const int64_t src = __shfl(row, r);
            const int e = e0 + c;
            dma4(X + src * d + (e < d ? e : d - 1), dst + 64 * i);
        }
    }
}
template <bool VEC> __device__ __forceinline__ f32x4 staged_vec(const float *s, int row, int c) {
    if constexpr (VEC)
        return *reinterpret_cast<const f32x4 *>(s + row * XB + 4 * (c ^ ((row >> 1) & 7)));
    f32x4 v;
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = s[row * XB + ((4 * c + q) ^ (row & 31))];
    return v;
}
// The exact value (ip64's arithmetic, term by term) of every lane's item row
// (prow, staged in sp) and user row: row myr of the nu rows of U that lanes 0,
// 1, ... name (urow), staged in ul, or (ONE) the one row ul of all lanes, in
// LDS, 16-byte aligned.
template <bool VEC, bool ONE>
__device__ __forceinline__ double ip64_rows(const float *P, int prow, int nrows, const float *U,
                                            int urow, int nu, int myr, float *ul, int d, float *sp,
                                            int lane) {
    double acc = 0.0;
    for (int e0 = 0; e0 < d; e0 += XB) {
        // the reads of the previous block are done before its place is written
        __builtin_amdgcn_s_waitcnt(0xc07f);  // (LDS operations only)
        wave_sync();
        stage_rows<VEC>(P, prow, nrows, d, e0, sp, lane);
        if constexpr (!ONE) stage_rows<VEC>(U, urow, nu, d, e0, ul, lane);
        dma_wait();
        wave_sync();
        const int left = d - e0;
#pragma unroll
        for (int c = 0; c < XB / 4; ++c) {
            if (4 * c >= left) break;
            const f32x4 y = staged_vec<VEC>(sp, lane, c);
            f32x4 x;
            if constexpr (ONE) x = *reinterpret_cast<const f32x4 *>(ul + e0 + 4 * c);
            else x = staged_vec<VEC>(ul, myr, c);
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (VEC || 4 * c + q < left) acc = __fma_rn((double)x[q], (double)y[q], acc);
        }
    }
    return acc;
}
__device__ __forceinline__ bool rows_vec(const float *U, const float *P, int d) {
    return (d & 3) == 0 &&
           ((reinterpret_cast<uintptr_t>(U) | reinterpret_cast<uintptr_t>(P)) & 15) == 0;
}

// The recomputations left by the selection, users with at most EXACT_SLOTS
// values: a wave takes 64 users of the list, joins their values and computes
// 64 of them at a time, one per lane; then lane u ranks user u's values: the
// one of rank tgt in the order (value desc, id asc) is tau_u.  2M users x 200
// with one value each 0.66 ms (8 lanes and their own loads per user: 1.45 ms).
constexpr int EXACT_WAVES = 2;  // per workgroup (LDS: 24 KB per wave)
__global__ __launch_bounds__(64 * EXACT_WAVES) void k_thresh_exact(ThreshArgs a) {
    __shared__ __align__(16) float sp_s[EXACT_WAVES][XB_FLOATS], su_s[EXACT_WAVES][XB_FLOATS];
    __shared__ double val_s[EXACT_WAVES][64 * EXACT_SLOTS];
    __shared__ int id_s[EXACT_WAVES][64 * EXACT_SLOTS];
    __shared__ uint8_t own_s[EXACT_WAVES][64 * EXACT_SLOTS];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int64_t nlist = (int64_t)*a.ulist_cnt;
    const int64_t capU = (int64_t)a.nsplit * a.cap;
    double *val = val_s[w];
    int *ids = id_s[w];
    uint8_t *own = own_s[w];
    const bool vec = rows_vec(a.U, a.P, a.d);
    for (int64_t b0 = ((int64_t)blockIdx.x * EXACT_WAVES + w) * 64; b0 < nlist;
         b0 += (int64_t)gridDim.x * EXACT_WAVES * 64) {
        const int64_t pos = b0 + lane;
        int u = 0, meta = -1;
        if (pos < nlist) {
            u = a.ulist[pos];
            meta = a.cand_cnt[(int64_t)u * a.nsplit];
        }
        // (longer lists are k_thresh_exact_wide's)
        const int nrec = (meta < 0 || (meta >> 8) > EXACT_SLOTS) ? 0 : meta >> 8;
        int off = nrec;  // inclusive prefix
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int y = __shfl_up(off, o);
            if (lane >= o) off += y;
        }
        const int total = __builtin_amdgcn_readlane(off, 63);
        off -= nrec;
        wave_sync();  // the previous users' lists are no longer read
        for (int q = 0; q < nrec; ++q) {
            ids[off + q] = a.cand_id[(int64_t)u * capU + q];
            own[off + q] = (uint8_t)lane;
        }
        wave_sync();
        for (int e0 = 0; e0 < total; e0 += 64) {
            const int e = e0 + lane;
            const int id = e < total ? ids[e] : 0;
            // the users of these values: lanes o0 .. o0 + nu - 1
            const int le = min(e0 + 63, total - 1);
            const int o0 = __builtin_amdgcn_readfirstlane((int)own[e0]);
            const int nu = __builtin_amdgcn_readfirstlane((int)own[le]) - o0 + 1;
            const int ur = __shfl(u, min(o0 + lane, 63));
            const int myr = (e < total ? own[e] : o0) - o0;
            const int nr = total - e0;
            const double v =
                vec ? ip64_rows<true, false>(a.P, id, nr, a.U, ur, nu, myr, su_s[w], a.d, sp_s[w], lane)
                    : ip64_rows<false, false>(a.P, id, nr, a.U, ur, nu, myr, su_s[w], a.d, sp_s[w], lane);
            if (e < total) val[e] = v;
        }
        wave_sync();
        const int tgt = meta & 255;
        for (int q = 0; q < nrec; ++q) {
            const double v = val[off + q];
            const int id = ids[off + q];
            int rank = 0;
            for (int j = 0; j < nrec; ++j) {
                const double y = val[off + j];
                rank += (y > v || (y == v && ids[off + j] < id)) ? 1 : 0;
            }
            if (rank == tgt) {
                a.tau[u] = v;
                a.tau_id[u] = id;
            }
            if (a.topk && rank < a.k) a.topk[(int64_t)u * a.k + rank] = id;
            if (a.topv && rank < a.k) a.topv[(int64_t)u * a.k + rank] = v;
        }
    }
}

// Sort key of a double (ascending; the sums never are -0 or NaN here).
__device__ __forceinline__ uint64_t double_key(double x) {
    const uint64_t b = (uint64_t)__double_as_longlong(x);
    return (b >> 63) ? ~b : (b | 0x8000000000000000ull);
}
__device__ __forceinline__ double key_double(uint64_t k) {
    return __longlong_as_double((long long)((k >> 63) ? (k & 0x7fffffffffffffffull) : ~k));
}
// The value of rank tgt (from 0) in the order (value desc, id asc) among the
// wave's values, J per lane (key 0: none): the largest key that tgt + 1 keys
// reach, bit by bit as in wave_kth_key, then the ids of the keys equal to it.
template <int J>
__device__ __forceinline__ void wave_rank64(const uint64_t (&r)[J], const int (&id)[J], int tgt,
                                            double &v, int &vid) {
    uint64_t t = 0;
    int above = 0;  // keys larger than the answer
    for (int b = 63; b >= 0; --b) {
        const uint64_t c = t | (1ull << b);
        int cnt = 0;
#pragma unroll
        for (int j = 0; j < J; ++j) cnt += __popcll(__ballot(r[j] >= c));
        if (cnt > tgt) t = c;
        else above = cnt;
        if (cnt == tgt + 1) {
            // exactly tgt + 1 keys: the smallest of them
            uint64_t m = ~0ull;
#pragma unroll
            for (int j = 0; j < J; ++j) m = r[j] >= c ? min(m, r[j]) : m;
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) m = min(m, (uint64_t)__shfl_xor((unsigned long long)m, o));
            t = m;
            int eq = 0;
#pragma unroll
            for (int j = 0; j < J; ++j) eq += __popcll(__ballot(r[j] == t));
            above = tgt + 1 - eq;
            break;
        }
    }
    v = key_double(t);
    // the (tgt - above)-th smallest id among the keys equal to t
    int last = -1;
    for (int q = above; q <= tgt; ++q) {
        int m = 0x7fffffff;
#pragma unroll
        for (int j = 0; j < J; ++j) m = (r[j] == t && id[j] > last) ? min(m, id[j]) : m;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) m = min(m, __shfl_xor(m, o));
        last = m;
    }
    vid = last;
}

// The recomputations of users with more than wide_from (EXACT_SLOTS, or 0
// where k_thresh_exact is left out) and at most EXACT_WIDE values: a wave per user, 64 values at a time (the user's row in LDS, the item
// rows through stage_rows), more than 64 by way of the user's candidate slots;
// tau_u by wave_rank64.  Each wave reads the metadata of its share of the list
// (at most 64 users at a time) and takes the wide ones in turn.  500k users x
// 100 with 156 values each 3.7 ms (each lane its own loads, the rank by rounds
// of maxima: 6.9 ms).
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4)))
void k_thresh_exact_wide(ThreshArgs a) {
    __shared__ __align__(16) float sp_s[4][XB_FLOATS];
    __shared__ __align__(16) float urow_s[4][DMAX];
    __shared__ double topv_s[4][KMAX];
    __shared__ int topi_s[4][KMAX];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int64_t nlist = (int64_t)*a.ulist_cnt;
    const int64_t capU = (int64_t)a.nsplit * a.cap;
    float *ul = urow_s[w], *sp = sp_s[w];
    const bool vec = rows_vec(a.U, a.P, a.d);
    // users of a wave at a time: few when the list is short, so that it
    // spreads over all waves
    const int64_t waves = (int64_t)gridDim.x * 4;
    const int per = (int)min<int64_t>(64, max<int64_t>(1, (nlist + waves - 1) / waves));
    for (int64_t c0 = ((int64_t)blockIdx.x * 4 + w) * per; c0 < nlist; c0 += waves * per) {
        const int64_t pos = c0 + lane;
        int myu = 0, meta = -1;
        if (lane < per && pos < nlist) {
            myu = a.ulist[pos];
            meta = a.cand_cnt[(int64_t)myu * a.nsplit];
        }
        uint64_t wide = __ballot(meta >= 0 && (meta >> 8) > a.wide_from);
        while (wide != 0ull) {
            const int src = __builtin_ctzll(wide);
            wide &= wide - 1ull;
            const int64_t u = __builtin_amdgcn_readlane(myu, src);
            const int mt = __builtin_amdgcn_readlane(meta, src);
            const int nrec = mt >> 8, tgt = mt & 255;
            const int32_t *ids = a.cand_id + u * capU;
            double *slots = reinterpret_cast<double *>(a.cand + u * capU);
            const float *urow = a.U + u * a.d;
            wave_sync();  // the previous user's row is no longer read
            for (int i = lane; i < a.d; i += 64) ul[i] = urow[i];
            wave_sync();
            double v = 0.0;
            int id = 0;
            for (int q0 = 0; q0 < nrec; q0 += 64) {
                const int q = q0 + lane;
                id = q < nrec ? ids[q] : 0;
                v = vec ? ip64_rows<true, true>(a.P, id, nrec - q0, nullptr, 0, 0, 0, ul, a.d, sp, lane)
                        : ip64_rows<false, true>(a.P, id, nrec - q0, nullptr, 0, 0, 0, ul, a.d, sp, lane);
                if (nrec > 64 && q < nrec) slots[q] = v;
            }
            double tv;
            int ti;
            // (each lane reads back only the values it wrote)
            auto rank_of = [&](auto jc) {
                constexpr int J = decltype(jc)::value;
                uint64_t r[J];
                int ri[J];
#pragma unroll
                for (int j = 0; j < J; ++j) {
                    const int q = lane + 64 * j;
                    r[j] = q < nrec ? double_key(J == 1 ? v : slots[q]) : 0ull;
                    ri[j] = q < nrec ? (J == 1 ? id : ids[q]) : 0x7fffffff;
                }
                wave_rank64(r, ri, tgt, tv, ti);
            };
            if (nrec <= 64) {
                rank_of(std::integral_constant<int, 1>{});
            } else if (nrec <= 256) {
                rank_of(std::integral_constant<int, 4>{});
            } else if (nrec <= EXACT_REGS) {
                rank_of(std::integral_constant<int, EXACT_REGS / 64>{});
            } else {
                // (rare) rounds of the next value in the order
                tv = INFINITY;
                ti = -1;
                for (int r = 0; r <= tgt; ++r) {
                    double bv = -INFINITY;
                    int bi = 0x7fffffff;
                    for (int q = lane; q < nrec; q += 64) {
                        const double x = slots[q];
                        const int xi = ids[q];
                        if ((x < tv || (x == tv && xi > ti)) && (x > bv || (x == bv && xi < bi))) {
                            bv = x;
                            bi = xi;
                        }
                    }
#pragma unroll
                    for (int o = 32; o > 0; o >>= 1) {
                        const double ov = __shfl_xor(bv, o);
                        const int oi = __shfl_xor(bi, o);
                        if (ov > bv || (ov == bv && oi < bi)) {
                            bv = ov;
                            bi = oi;
                        }
                    }
                    tv = bv;
                    ti = bi;
                }
            }
            if (a.topk) {
                // the k values up to tau in the order (tgt = k - 1), then
                // their places among themselves
                int nt = 0;
                for (int q0 = 0; q0 < nrec; q0 += 64) {
                    const int q = q0 + lane;
                    const double x = q < nrec ? (nrec > 64 ? slots[q] : v) : -INFINITY;
                    const int xi = q < nrec ? ids[q] : 0x7fffffff;
                    const bool in = q < nrec && (x > tv || (x == tv && xi <= ti));
                    const uint64_t bal = __ballot(in);
                    const int p = nt + __popcll(bal & ((lane == 0) ? 0ull : (~0ull >> (64 - lane))));
                    if (in) {
                        topv_s[w][p] = x;
                        topi_s[w][p] = xi;
                    }
                    nt += __popcll(bal);
                }
                wave_sync();
                if (lane < a.k) {
                    const double x = topv_s[w][lane];
                    const int xi = topi_s[w][lane];
                    int rank = 0;
                    for (int j = 0; j < a.k; ++j) {
                        const double y = topv_s[w][j];
                        rank += (y > x || (y == x && topi_s[w][j] < xi)) ? 1 : 0;
                    }
                    a.topk[u * a.k + rank] = xi;
                    if (a.topv) a.topv[u * a.k + rank] = x;
                }
                wave_sync();
            }
            if (lane == 0) {
                a.tau[u] = tv;
                a.tau_id[u] = ti;
            }
        }
    }
}

// ------------------------------------------------------------------ fallback
// Brute force for users whose candidate list overflowed: one wave per user,
// every item in FP64, per-lane top-k lists merged by k rounds of a wave-wide
// maximum under (value desc, id asc).
constexpr int FB_WAVES = 2;

__global__ __launch_bounds__(64 * FB_WAVES) void k_thresh_fallback(ThreshArgs a) {
    __shared__ double lv[FB_WAVES][64][KMAX];
    __shared__ int li[FB_WAVES][64][KMAX];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int k = a.k;
    const int64_t nf = *a.fcnt;
    for (int64_t i = (int64_t)blockIdx.x * FB_WAVES + w; i < nf;
         i += (int64_t)gridDim.x * FB_WAVES) {
        const int64_t u = a.flist[i];
        const float *urow = a.U + u * a.d;
        double *myv = lv[w][lane];
        int *myi = li[w][lane];
        int cnt = 0;
        for (int64_t j = lane; j < a.m; j += 64) {
            const int c = (int)j;  // caller id
            const double v = ip64(urow, a.P + j * a.d, a.d);
            if (cnt == k) {
                const double tv = myv[k - 1];
                const int ti = myi[k - 1];
                if (!(v > tv || (v == tv && c < ti))) continue;
            }
            int pos = (cnt < k) ? cnt : k - 1;
            while (pos > 0 && (myv[pos - 1] < v || (myv[pos - 1] == v && myi[pos - 1] > c))) {
                myv[pos] = myv[pos - 1];
                myi[pos] = myi[pos - 1];
                --pos;
            }
            myv[pos] = v;
            myi[pos] = c;
            if (cnt < k) ++cnt;
        }
        int head = 0;
        for (int r = 0; r < k; ++r) {
            double bv = (head < cnt) ? myv[head] : -INFINITY;
            int bi = (head < cnt) ? myi[head] : 0x7fffffff;
            int bl = lane;
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) {
                double ov = __shfl_xor(bv, o);
                int oi = __shfl_xor(bi, o);
                int ol = __shfl_xor(bl, o);
                if (ov > bv || (ov == bv && oi < bi)) {
                    bv = ov;
                    bi = oi;
                    bl = ol;
                }
            }
            if (lane == bl) ++head;
            if (lane == 0) {
                if (a.topk) a.topk[u * k + r] = bi;
                if (a.topv) a.topv[u * k + r] = bv;
                if (r == k - 1) {
                    a.tau[u] = bv;
                    a.tau_id[u] = bi;
                }
            }
        }
    }
}

template <int PREC>
void launch_screen(const ThreshArgs &a, int nch, dim3 g, size_t lds, hipStream_t st,
                   const char *name) {
    RMIPS_PROF(st, name);
    with_nch<PREC>(nch, [&](auto n) {
        constexpr int NCH = decltype(n)::value;
        if constexpr (screen_u2(PREC, NCH)) {
            if (a.ulist) {
                k_thresh_screen_u2<PREC, NCH><<<g, 64 * SCR2_NW, lds, st>>>(a);
                return;
            }
        }
        if (a.ulist) k_thresh_screen<PREC, NCH, true><<<g, 64 * screen_nw<true>(PREC, NCH), lds, st>>>(a);
        else k_thresh_screen<PREC, NCH, false><<<g, 64 * screen_nw<false>(PREC, NCH), lds, st>>>(a);
    });
}

// Sort keys of the users' early-exit ratios (ascending): the norm below
// which no item reaches the user's starting bound, as in the screening
// kernel; users whose bound is not positive scan every tile (ratio 0).
__global__ void k_exit_keys(ThreshArgs a, uint32_t *__restrict__ key, int32_t *__restrict__ val) {
    const int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (u == 0) {  // the list counters of the passes that follow
        a.lcnt[0] = 0;
        a.lcnt[1] = 0;
        a.lcnt[2] = 0;
        a.lcnt[3] = 0;
        *a.nall = (int32_t)a.n;  // the main pass takes every user
    }
    if (u >= a.n) return;
    const float rmax = __uint_as_float(*a.rmax_bits);
    const float nu = a.Nu[u], nhu = a.Nhu[u], ru = a.Ru[u], L = a.Luse[u];
    const float K = nu * (1.0f + a.g64 + 2.0f * a.c2) + 2.0f * ru +
                    2.0f * nhu * (rmax + a.c_err * (1.0f + rmax));
    const float rr = (L > 2.0f * a.e_abs && K > 0.0f) ? (L - 2.0f * a.e_abs) / K : 0.0f;
    key[u] = float_key(rr);
    val[u] = (int32_t)u;
}

void launch_thresh(const ThreshArgs &a0, hipStream_t st) {
    const int nch = a0.D * elem_bytes(a0.prec) / 32;
    // users per workgroup of the passes with a user list
    const int tu = screen_u2(a0.prec, nch) ? 64 * SCR2_NW : 32 * screen_waves(a0.prec, nch);
    const size_t lds = thresh_screen_lds(a0.prec, a0.D);
    const int64_t ublocks = (a0.n + tu - 1) / tu;
    const int capU = a0.cap * a0.nsplit;
    const int capP = final_stride(capU);
    int fw = (int)((150 * 1024) / ((size_t)capP * FIN_ENTRY_BYTES));  // waves whose lists fit in LDS
    fw = fw < 1 ? 1 : (fw > FIN_WAVES ? FIN_WAVES : fw);
    const size_t lds_fin = (size_t)fw * capP * FIN_ENTRY_BYTES;
    // one resident round of workgroups (FIN_WPE per CU, fewer when their
    // lists fill the LDS): each wave takes many users in turn
    const int64_t fres =
        256 * std::max<int64_t>(1, std::min<int64_t>(FIN_WPE * 4 / fw, (160 * 1024) / lds_fin));
    const int64_t fblocks = std::min<int64_t>((a0.n + fw - 1) / fw, fres);
    // (a wave per 64 users; three 2-wave workgroups per CU are resident)
    const int64_t eblocks = std::min<int64_t>((a0.n + 64 * EXACT_WAVES - 1) / (64 * EXACT_WAVES), 6 * 256);
    // one resident round (four 4-wave workgroups per CU)
    constexpr int64_t wblocks_max = 4 * 256;
    const int64_t wblocks = std::min<int64_t>((a0.n + 3) / 4, wblocks_max);
    int32_t *LA = a0.lists, *LB = a0.lists + a0.n, *LF = a0.lists + 2 * a0.n;
    auto screen = [&](const ThreshArgs &a, dim3 g, const char *name) {
        if (a.prec == PREC_FP32) launch_screen<PREC_FP32>(a, nch, g, lds, st, name);
        else if (a.prec == PREC_SPLIT) launch_screen<PREC_SPLIT>(a, nch, g, lds, st, name);
        else if (a.prec == PREC_BF16) launch_screen<PREC_BF16>(a, nch, g, lds, st, name);
        else if (a.prec == PREC_FP8) launch_screen<PREC_FP8>(a, nch, g, lds, st, name);
        else if (a.prec == PREC_FP6) launch_screen<PREC_FP6>(a, nch, g, lds, st, name);
        else launch_screen<PREC_FP4>(a, nch, g, lds, st, name);
    };
    // the screening pass writes each (user, split) list as two halves of
    // cap / 2 entries with their own counts: the final selection and the
    // deferred recomputations read them as 2 * nsplit lists
    auto final = [&](const ThreshArgs &a, int capT, const char *ns, const char *nf,
                     const char *ne, const char *nw) {
        ThreshArgs h = a;
        h.nsplit = 2 * a.nsplit;
        h.cap = a.cap / 2;
        if (capT <= SEL_MAX) {
            RMIPS_PROF(st, ns);
            auto select = [&](auto mx) {
                constexpr int MAX = decltype(mx)::value;
                // one resident round: a 4-wave workgroup per wave of a SIMD
                const int64_t sblocks = std::min<int64_t>((a0.n + 3) / 4, 256 * sel_waves(MAX));
                k_thresh_select<MAX><<<(unsigned)sblocks, 256, 0, st>>>(h);
            };
            if (capT <= SEL_SHORT) select(std::integral_constant<int, SEL_SHORT>{});
            else if (capT <= SEL_MID) select(std::integral_constant<int, SEL_MID>{});
            else select(std::integral_constant<int, SEL_MAX>{});
        } else {
            RMIPS_PROF(st, nf);
            k_thresh_final<<<(unsigned)fblocks, 64 * fw, lds_fin, st>>>(h, capT, capP);
        }
        // A launch costs about 5 us whatever it does.  The refinement passes'
        // lists are empty or hold many values, and up to 4096 users find a
        // wave each: there k_thresh_exact_wide takes all lists (2000 users x
        // 1000 items: the call 293 -> 274 us together with k_user_order)
        h.wide_from = a.n <= 4 * wblocks_max || ne == nullptr ? 0 : EXACT_SLOTS;
        if (h.wide_from > 0) {
            RMIPS_PROF(st, ne);
            k_thresh_exact<<<(unsigned)eblocks, 64 * EXACT_WAVES, 0, st>>>(h);
        }
        RMIPS_PROF(st, nw);
        k_thresh_exact_wide<<<(unsigned)wblocks, 256, 0, st>>>(h);
    };
    // bounds-only pass (the launch without a user list): every user's L0
    // from the first tiles (phase 1), in workgroups of its own size
    ThreshArgs b0 = a0;
    b0.ulist = nullptr;
    b0.ulist_cnt = nullptr;
    b0.nsplit = 1;
    b0.pairs = nullptr;
    const int tu1 = 32 * screen_waves_p1(a0.prec, nch);
    screen(b0, dim3((unsigned)((a0.n + tu1 - 1) / tu1), 1u), "k_thresh_screen/bounds");
    // users in the order of their early-exit ratios, so that the users of a
    // workgroup stop their scans at about the same tile
    {
        RMIPS_PROF(st, "k_exit_keys");
        k_exit_keys<<<(unsigned)((a0.n + 255) / 256), 256, 0, st>>>(a0, a0.ukey, a0.uord);
    }
    // a grouping only: the top 16 bits of the ratio (sign, exponent and 7
    // mantissa bits) are enough, ties stay in user order
    (void)radix_sort_u32(a0.ukey, a0.uord, a0.n, a0.usort, st, 16, 32);
    // main pass: all users, in that order, from their L0
    ThreshArgs a = a0;
    a.ulist = a0.uord;
    a.ulist_cnt = a0.nall;
    a.rlist = a0.refine > 0 ? LA : nullptr;
    a.rcnt = a0.lcnt;
    a.flist = LF;
    a.fcnt = a0.lcnt + 2;
    if (a.ev0) (void)hipEventRecord(a.ev0, st);
    screen(a, dim3((unsigned)ublocks, (unsigned)a.nsplit), "k_thresh_screen/main");
    if (a.ev1) (void)hipEventRecord(a.ev1, st);
    final(a, capU, "k_thresh_select/main", "k_thresh_final/main", "k_thresh_exact/main",
          "k_thresh_exact_wide/main");
    // refinement passes over the users whose lists overflowed: the same
    // per-user capacity in fewer, longer lists per split
    int nsr = capU / 64;
    nsr = nsr < 1 ? 1 : (nsr > 8 ? 8 : nsr);
    for (int r = 1; r <= a0.refine && r <= 2; ++r) {
        ThreshArgs b = a0;
        b.ulist = (r == 1) ? LA : LB;
        b.ulist_cnt = a0.lcnt + (r == 1 ? 0 : 1);
        b.rlist = (r < a0.refine && r < 2) ? LB : nullptr;
        b.rcnt = a0.lcnt + 1;
        b.flist = LF;
        b.fcnt = a0.lcnt + 2;
        b.nsplit = nsr;
        b.cap = (capU / nsr) & ~1;  // (even: two halves per list)
        b.t0tiles = 0;
        b.pairs = a0.rpairs;
        // one resident round (one screening workgroup per CU): the lists
        // are usually empty, and the workgroups loop over long ones
        const int64_t gx = ublocks < 256 / nsr ? ublocks : 256 / nsr;
        screen(b, dim3((unsigned)gx, (unsigned)nsr), "k_thresh_screen/refine");
        final(b, b.nsplit * b.cap, "k_thresh_select/refine", "k_thresh_final/refine", nullptr,
              "k_thresh_exact_wide/refine");
    }
    int64_t fb = (a0.n + FB_WAVES - 1) / FB_WAVES;
    if (fb > 1024) fb = 1024;
    a.flist = LF;
    a.fcnt = a0.lcnt + 2;
    RMIPS_PROF(st, "k_thresh_fallback");
    k_thresh_fallback<<<(unsigned)fb, 64 * FB_WAVES, 0, st>>>(a);
}

}  // namespace rmips
