// Stable LSD radix sort of (uint32 key, int32 value) pairs, 8 bits per pass.
//
// Used for the orderings the method needs: items by norm (descending),
// users by their pruning ratio tau_u/||u||, and items by upper-bound score
// (descending) with ties kept in item-id order.  Stability is what carries
// the id tie order through: inputs are laid out in id order.
#include "common.h"
#include "kernels.h"

namespace rmips {

constexpr int SORT_THREADS = 256;
// Up to this many blocks a pass needs no scan kernels: every scatter block
// sums the digit counts of all blocks itself.  Counts of a pass are then
// laid out [block][digit], otherwise [digit][block] (scanned in place).
constexpr int PREFIX_MAX_BLOCKS = 128;
// Elements per block: 256 x 4, or 256 x 16 where that, and not 256 x 4, keeps a
// pass at that many blocks (500k keys: 122 blocks of 4,096 and no scans, 33 us a
// pass, against 488 blocks and 45 us with the scans).  Longer lists take scans
// either way, and the smaller blocks then fill the chip better (2M keys: 0.09
// against 0.2 ms a pass).
constexpr int SORT_R_SMALL = 4, SORT_R_LARGE = 16;
inline int sort_rounds(int64_t n) {
    const int64_t one = (int64_t)PREFIX_MAX_BLOCKS * SORT_THREADS;
    return n > one * SORT_R_SMALL && n <= one * SORT_R_LARGE ? SORT_R_LARGE : SORT_R_SMALL;
}
// Up to BLOCK_SORT elements one workgroup sorts alone, every pass in LDS: one
// launch instead of one per pass and one for the counts (2,000 keys: four sorts
// of 16 to 32 bits 38 us, against 130 us in 15 launches).
constexpr int BLOCK_SORT = 8192, BLOCK_SORT_THREADS = 1024;

// Lanes of this wave (of those in `act`) that hold the same digit as this one.
__device__ __forceinline__ uint64_t digit_peers(uint64_t act, uint32_t dig) {
    uint64_t peers = act;
#pragma unroll
    for (int b = 0; b < 8; ++b) {
        const uint64_t bb = __ballot((dig >> b) & 1u);
        peers &= ((dig >> b) & 1u) ? bb : ~bb;
    }
    return peers;
}
// Orders a wave's own LDS accesses.
__device__ __forceinline__ void sort_wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}
// Ranks of a wave's elements among those of the wave with the same digit, in
// element order (round r, lane l: element 64 r + l): cnt[dig] counts the rounds
// before (LDS, one row per wave, cleared before).
template <int R>
__device__ __forceinline__ void wave_digit_ranks(const uint32_t (&dig)[R], const bool (&act)[R],
                                                 uint32_t *cnt, uint64_t lt, uint32_t (&rank)[R],
                                                 uint64_t (&peers)[R]) {
#pragma unroll
    for (int r = 0; r < R; ++r) {
        peers[r] = digit_peers(__ballot(act[r]), dig[r]);
        const uint32_t in = __popcll(peers[r] & lt);
        const uint32_t before = act[r] ? cnt[dig[r]] : 0u;
        rank[r] = before + in;
        sort_wave_sync();
        if (act[r] && in == 0) cnt[dig[r]] = before + (uint32_t)__popcll(peers[r]);
        sort_wave_sync();
    }
}

__device__ __forceinline__ int64_t count_index(bool small, uint32_t dig, int64_t blk,
                                               int nblocks) {
    return small ? blk * 256 + dig : (int64_t)dig * nblocks + blk;
}

// Digit counts of the first pass per block; clears the counts of the later
// passes, which the scatter of the pass before each of them accumulates.
template <int R>
__global__ __launch_bounds__(SORT_THREADS) void k_radix_hist(
    const uint32_t *__restrict__ keys, int64_t n, int shift, int nblocks, int npass,
    uint32_t *__restrict__ counts) {
    __shared__ uint32_t hist[256];
    const int t = threadIdx.x;
    const bool small = nblocks <= PREFIX_MAX_BLOCKS;
    hist[t] = 0;
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * (SORT_THREADS * R);
    uint32_t kr[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int64_t e = base + (int64_t)r * SORT_THREADS + t;
        kr[r] = e < n ? keys[e] : 0u;
    }
#pragma unroll
    for (int r = 0; r < R; ++r)
        if (base + (int64_t)r * SORT_THREADS + t < n) atomicAdd(&hist[(kr[r] >> shift) & 255u], 1u);
    __syncthreads();
    const int64_t stride = (int64_t)256 * nblocks;
    const int64_t ci = count_index(small, t, blockIdx.x, nblocks);
    counts[ci] = hist[t];
    for (int q = 1; q < npass; ++q) counts[q * stride + ci] = 0;
}

// Exclusive scan of counts[0, total) in place, in tiles of SCAN_TILE
// entries: the first kernel sums each tile, the second scans each tile from
// the sum of the tiles before it (at most a few dozen, read by every block).
constexpr int SCAN_PER_THREAD = 16;
constexpr int SCAN_TILE = SORT_THREADS * SCAN_PER_THREAD;

__global__ __launch_bounds__(SORT_THREADS) void k_scan_reduce(const uint32_t *__restrict__ counts,
                                                              int64_t total,
                                                              uint32_t *__restrict__ tsum) {
    __shared__ uint32_t ws[SORT_THREADS / WAVE];
    const int t = threadIdx.x;
    const int64_t b0 = (int64_t)blockIdx.x * SCAN_TILE;
    uint32_t s = 0;
#pragma unroll
    for (int r = 0; r < SCAN_PER_THREAD; ++r) {
        const int64_t e = b0 + (int64_t)r * SORT_THREADS + t;
        s += (e < total) ? counts[e] : 0u;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
    if ((t & 63) == 0) ws[t >> 6] = s;
    __syncthreads();
    if (t == 0) {
        uint32_t x = 0;
        for (int q = 0; q < SORT_THREADS / WAVE; ++q) x += ws[q];
        tsum[blockIdx.x] = x;
    }
}

__global__ __launch_bounds__(SORT_THREADS) void k_scan_down(uint32_t *__restrict__ counts,
                                                            int64_t total,
                                                            const uint32_t *__restrict__ tsum) {
    __shared__ uint32_t tot[SORT_THREADS];
    __shared__ uint32_t base;
    const int t = threadIdx.x;
    if (t == 0) {
        uint32_t x = 0;
        for (int q = 0; q < (int)blockIdx.x; ++q) x += tsum[q];
        base = x;
    }
    // each thread: SCAN_PER_THREAD consecutive entries
    const int64_t e0 = (int64_t)blockIdx.x * SCAN_TILE + (int64_t)t * SCAN_PER_THREAD;
    uint32_t v[SCAN_PER_THREAD];
    uint32_t s = 0;
#pragma unroll
    for (int r = 0; r < SCAN_PER_THREAD; ++r) {
        v[r] = (e0 + r < total) ? counts[e0 + r] : 0u;
        s += v[r];
    }
    tot[t] = s;
    __syncthreads();
    // inclusive scan of the thread sums
    for (int o = 1; o < SORT_THREADS; o <<= 1) {
        const uint32_t y = (t >= o) ? tot[t - o] : 0u;
        __syncthreads();
        tot[t] += y;
        __syncthreads();
    }
    uint32_t run = base + tot[t] - s;
#pragma unroll
    for (int r = 0; r < SCAN_PER_THREAD; ++r) {
        if (e0 + r < total) counts[e0 + r] = run;
        run += v[r];
    }
}

// One pass: block b moves its 256 R elements to their places (wave w the 64 R
// from w * 64 R on).  Its
// first output slot per digit comes either from the scanned counts, or
// (small) from summing the counts of all blocks here: digits before this one
// over all blocks, plus this digit over the blocks before b.  With nshift >=
// 0 the pass also counts the next pass's digits per destination block.
template <int R>
__global__ __launch_bounds__(SORT_THREADS) void k_radix_scatter(
    const uint32_t *__restrict__ kin, const int32_t *__restrict__ vin,
    uint32_t *__restrict__ kout, int32_t *__restrict__ vout, int64_t n,
    int shift, int nshift, int nblocks, const uint32_t *__restrict__ counts,
    uint32_t *__restrict__ cnext) {
    __shared__ uint32_t base[256];
    __shared__ uint32_t wcnt[SORT_THREADS / WAVE][256];
    __shared__ uint32_t ptot[SORT_THREADS / WAVE][256];
    __shared__ uint32_t wsum[SORT_THREADS / WAVE];
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    const bool small = nblocks <= PREFIX_MAX_BLOCKS;
    // this thread's elements of all rounds, loaded before the offsets are
    // summed
    constexpr int CHUNK = SORT_THREADS * R;
    const int64_t b0 = (int64_t)blockIdx.x * CHUNK + w * 64 * R + lane;
    uint32_t kr[R], dig[R];
    int32_t vr[R];
    bool act[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int64_t e = b0 + 64 * r;
        act[r] = e < n;
        kr[r] = act[r] ? kin[e] : 0u;
        vr[r] = act[r] ? vin[e] : 0;
        dig[r] = (kr[r] >> shift) & 255u;
    }
    if (small) {
        // wave w sums the rows w, w + 4, ...: lane l holds digits 4l..4l+3;
        // wcnt collects the rows before this block, ptot all rows
        const uint4 *c4 = reinterpret_cast<const uint4 *>(counts);
        uint4 pre = make_uint4(0, 0, 0, 0), tot = make_uint4(0, 0, 0, 0);
#pragma unroll 8
        for (int b = w; b < nblocks; b += SORT_THREADS / WAVE) {
            const uint4 c = c4[(int64_t)b * 64 + lane];
            tot.x += c.x; tot.y += c.y; tot.z += c.z; tot.w += c.w;
            if (b < (int)blockIdx.x) { pre.x += c.x; pre.y += c.y; pre.z += c.z; pre.w += c.w; }
        }
        reinterpret_cast<uint4 *>(&ptot[w][0])[lane] = tot;
        reinterpret_cast<uint4 *>(&wcnt[w][0])[lane] = pre;
        __syncthreads();
        uint32_t T = 0, P = 0;
#pragma unroll
        for (int q = 0; q < SORT_THREADS / WAVE; ++q) {
            T += ptot[q][t];
            P += wcnt[q][t];
        }
        // exclusive scan of the digit totals over the 256 digits
        uint32_t x = T;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t y = __shfl_up(x, o);
            if (lane >= o) x += y;
        }
        if (lane == 63) wsum[w] = x;
        __syncthreads();
        uint32_t before = 0;
        for (int q = 0; q < w; ++q) before += wsum[q];
        base[t] = before + x - T + P;
        for (int q = 0; q < SORT_THREADS / WAVE; ++q) wcnt[q][t] = 0;
    } else {
        base[t] = counts[count_index(false, t, blockIdx.x, nblocks)];
        for (int q = 0; q < SORT_THREADS / WAVE; ++q) wcnt[q][t] = 0;
    }
    __syncthreads();
    const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    uint32_t rank[R];
    uint64_t peers[R];
    wave_digit_ranks<R>(dig, act, wcnt[w], lt, rank, peers);
    __syncthreads();
    {
        // first slot of each wave's elements of digit t
        uint32_t run = base[t];
#pragma unroll
        for (int q = 0; q < SORT_THREADS / WAVE; ++q) {
            const uint32_t c = wcnt[q][t];
            wcnt[q][t] = run;
            run += c;
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const uint32_t off = wcnt[w][dig[r]] + rank[r];
        if (act[r]) {
            kout[off] = kr[r];
            vout[off] = vr[r];
        }
        if (nshift >= 0) {
            // the next digits per destination block: one atomic per group of
            // peers with the same next digit and block (a digit's peers of a
            // round fill consecutive slots, so they meet at most two blocks,
            // told apart by the block's lowest bit)
            const uint32_t nd = (kr[r] >> nshift) & 255u, db = off / CHUNK;
            uint64_t grp = digit_peers(peers[r], nd);
            const uint64_t bb = __ballot(db & 1u);
            grp &= (db & 1u) ? bb : ~bb;
            if (act[r] && (grp & lt) == 0ull)
                atomicAdd(&cnext[count_index(small, nd, db, nblocks)], (uint32_t)__popcll(grp));
        }
    }
}

// All passes of a short list in one workgroup: keys and values in registers,
// exchanged through LDS after each pass.  Wave w holds elements w * 64 R on.
constexpr size_t block_sort_lds(int R) {
    return (size_t)BLOCK_SORT_THREADS * R * 8 + (BLOCK_SORT_THREADS / WAVE + 1) * 256 * 4 + 64;
}
template <int R>
__global__ __launch_bounds__(BLOCK_SORT_THREADS) void k_block_sort(uint32_t *__restrict__ keys,
                                                                   int32_t *__restrict__ vals,
                                                                   int n, int lo_bit, int npass) {
    extern __shared__ uint32_t sort_lds[];
    constexpr int NWV = BLOCK_SORT_THREADS / WAVE;
    uint32_t *sk = sort_lds;
    int32_t *sv = reinterpret_cast<int32_t *>(sk + BLOCK_SORT_THREADS * R);
    uint32_t(*wcnt)[256] = reinterpret_cast<uint32_t(*)[256]>(sv + BLOCK_SORT_THREADS * R);
    uint32_t *wsum = &wcnt[NWV][0];
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    const int b0 = w * 64 * R + lane;
    uint32_t kr[R], dig[R], rank[R];
    uint64_t peers[R];
    int32_t vr[R];
    bool act[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int e = b0 + 64 * r;
        act[r] = e < n;
        kr[r] = act[r] ? keys[e] : 0u;
        vr[r] = act[r] ? vals[e] : 0;
    }
    for (int q = 0; q < npass; ++q) {
        const int shift = lo_bit + 8 * q;
        for (int i = t; i < NWV * 256; i += BLOCK_SORT_THREADS) (&wcnt[0][0])[i] = 0u;
#pragma unroll
        for (int r = 0; r < R; ++r) dig[r] = (kr[r] >> shift) & 255u;
        __syncthreads();
        wave_digit_ranks<R>(dig, act, wcnt[w], lt, rank, peers);
        __syncthreads();
        // digit t: counts before each wave, the total scanned over the digits
        uint32_t run = 0u, x = 0u;
        if (t < 256) {
            for (int v = 0; v < NWV; ++v) {
                const uint32_t c = wcnt[v][t];
                wcnt[v][t] = run;
                run += c;
            }
            x = run;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const uint32_t y = __shfl_up(x, o);
                if (lane >= o) x += y;
            }
            if (lane == 63) wsum[w] = x;
        }
        __syncthreads();
        if (t < 256) {
            uint32_t first = x - run;
            for (int v = 0; v < w; ++v) first += wsum[v];
            for (int v = 0; v < NWV; ++v) wcnt[v][t] += first;
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < R; ++r)
            if (act[r]) {
                const uint32_t off = wcnt[w][dig[r]] + rank[r];
                sk[off] = kr[r];
                sv[off] = vr[r];
            }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < R; ++r)
            if (act[r]) {
                kr[r] = sk[b0 + 64 * r];
                vr[r] = sv[b0 + 64 * r];
            }
    }
#pragma unroll
    for (int r = 0; r < R; ++r)
        if (act[r]) {
            keys[b0 + 64 * r] = kr[r];
            vals[b0 + 64 * r] = vr[r];
        }
}

// (enough for every shorter list too: those of 128 blocks of 1,024 and fewer
// take more blocks than some longer ones)
size_t radix_sort_scratch_bytes(int64_t n) {
    const int64_t chunk = (int64_t)SORT_THREADS * sort_rounds(n);
    const int64_t nblocks = std::max<int64_t>(
        std::max<int64_t>(1, (n + chunk - 1) / chunk),
        std::min<int64_t>(PREFIX_MAX_BLOCKS, n / (SORT_THREADS * SORT_R_SMALL) + 1));
    const int64_t ntiles = (256 * nblocks + SCAN_TILE - 1) / SCAN_TILE;
    return (size_t)(4 * 256 * nblocks) * sizeof(uint32_t) +
           2 * ((size_t)n * (sizeof(uint32_t) + sizeof(int32_t)) + 256) +
           (size_t)ntiles * 4 + 1024;
}

// Sort (keys, vals) ascending by the key bits [lo_bit, hi_bit), stably; the
// bits at and above hi_bit must be the same in every key (then the order is
// that of the whole keys).  8 bits per pass, the result in the input
// buffers; `scratch` holds radix_sort_scratch_bytes(n) bytes.
hipError_t radix_sort_u32(uint32_t *keys, int32_t *vals, int64_t n, void *scratch,
                          hipStream_t st, int lo_bit, int hi_bit) {
    if (n <= 1 || hi_bit <= lo_bit) return hipSuccess;
    if (lo_bit < 0 || hi_bit > 32) return hipErrorInvalidValue;
    int npass = (hi_bit - lo_bit + 7) / 8;
    if (n <= BLOCK_SORT) {
        RMIPS_PROF(st, "k_block_sort");
        auto go = [&](auto rc) {
            constexpr int R = decltype(rc)::value;
            k_block_sort<R><<<1, BLOCK_SORT_THREADS, block_sort_lds(R), st>>>(keys, vals, (int)n,
                                                                              lo_bit, npass);
        };
        if (n <= 1024) go(std::integral_constant<int, 1>{});
        else if (n <= 2048) go(std::integral_constant<int, 2>{});
        else if (n <= 4096) go(std::integral_constant<int, 4>{});
        else go(std::integral_constant<int, BLOCK_SORT / BLOCK_SORT_THREADS>{});
        return hipGetLastError();
    }
    // A pass of several blocks does not write where it reads: a block's writes
    // would meet elements that another has yet to load.  So a single pass is
    // followed by a second one on eight more bits (those above hi_bit, the same
    // in every key, or again the last eight): it keeps the order and brings the
    // result back.
    if (npass == 1) npass = 2;
    const int rounds = sort_rounds(n), chunk = SORT_THREADS * rounds;
    const int nblocks = (int)((n + chunk - 1) / chunk);
    const bool small = nblocks <= PREFIX_MAX_BLOCKS;
    const int64_t total = (int64_t)256 * nblocks;
    uint32_t *counts = (uint32_t *)scratch;
    uint8_t *p = (uint8_t *)scratch + (size_t)4 * total * sizeof(uint32_t);
    auto carve = [&](size_t bytes) {
        p = (uint8_t *)(((uintptr_t)p + 255) & ~(uintptr_t)255);
        uint8_t *q = p;
        p += bytes;
        return q;
    };
    uint32_t *k1 = (uint32_t *)carve((size_t)n * 4), *k2 = (uint32_t *)carve((size_t)n * 4);
    int32_t *v1 = (int32_t *)carve((size_t)n * 4), *v2 = (int32_t *)carve((size_t)n * 4);
    uint32_t *tsum = (uint32_t *)carve(0);
    const int ntiles = (int)((total + SCAN_TILE - 1) / SCAN_TILE);
    {
        RMIPS_PROF(st, "k_radix_hist");
        if (rounds == SORT_R_SMALL)
            k_radix_hist<SORT_R_SMALL><<<nblocks, SORT_THREADS, 0, st>>>(keys, n, lo_bit, nblocks,
                                                                         npass, counts);
        else
            k_radix_hist<SORT_R_LARGE><<<nblocks, SORT_THREADS, 0, st>>>(keys, n, lo_bit, nblocks,
                                                                         npass, counts);
    }
    // the passes run keys -> 1 -> 2 -> 1 ... and the last one writes keys
    const uint32_t *ks = keys;
    const int32_t *vs = vals;
    for (int q = 0; q < npass; ++q) {
        const int shift = std::min(lo_bit + 8 * q, 24);
        const bool last = q == npass - 1;
        uint32_t *kd = last ? keys : ((q & 1) ? k2 : k1);
        int32_t *vd = last ? vals : ((q & 1) ? v2 : v1);
        uint32_t *cq = counts + q * total;
        const int next = last ? -1 : std::min(lo_bit + 8 * (q + 1), 24);
        if (!small) {
            RMIPS_PROF(st, "k_scan");
            k_scan_reduce<<<ntiles, SORT_THREADS, 0, st>>>(cq, total, tsum);
            k_scan_down<<<ntiles, SORT_THREADS, 0, st>>>(cq, total, tsum);
        }
        RMIPS_PROF(st, "k_radix_scatter");
        if (rounds == SORT_R_SMALL)
            k_radix_scatter<SORT_R_SMALL><<<nblocks, SORT_THREADS, 0, st>>>(
                ks, vs, kd, vd, n, shift, next, nblocks, cq, cq + total);
        else
            k_radix_scatter<SORT_R_LARGE><<<nblocks, SORT_THREADS, 0, st>>>(
                ks, vs, kd, vd, n, shift, next, nblocks, cq, cq + total);
        ks = kd;
        vs = vd;
    }
    return hipGetLastError();
}

}  // namespace rmips
