// Transposition of interaction lists on gfx950: from the sources of each sink
// leaf to the sinks of each source cell, in ascending order of the sinks.
//
// The pairs (target, sink leaf), in the order of the lists, are sorted by
// target with a stable radix sort of one or two digits of 8 to 10 bits.  What
// bounds it is the traffic (1.6e8 pairs for the far lists of a Plummer sphere
// of 2^19 particles) and, per pair and pass, the ballots that rank equal digits:
//   - the first pass reads the lists themselves; a pair that leaves it is one
//     word, the target's high digit over the leaf index (the low digit is given
//     by the position from there on), and the second pass writes the sinks
//     alone: 24 bytes per pair;
//   - the digits are no wider than the targets need;
//   - the pairs' leaves come from a table of every 64th one, so that the loads
//     of a wavefront's rounds do not wait for searches;
//   - the offsets of the targets follow from the digit counts of the two
//     passes and a part of one tile per low digit.
// Far and near lists together, with the offsets: 2.6 ms for Plummer, 2^19
// particles, 0.40 ms for the binary, 2^19; with the pairs written out as
// (key, value), sorted on 10-bit digits and searched for the offsets (56 bytes
// per pair) 4.8 and 0.63 ms.  Tiles of 4096 pairs by 512 lanes leave four
// workgroups per CU: by 1024 lanes 3.0 and 0.42 ms, by 256 lanes 3.0 and 0.44;
// 8192 pairs 3.2 and 0.49.
#include "fmm_internal.h"

namespace fmm {

constexpr int TP_THREADS = 512, TP_WAVES = TP_THREADS / 64, TP_ROUNDS = 8;
constexpr int TP_TILE = TP_THREADS * TP_ROUNDS;
constexpr int TP_SEG = 64;  // pairs per entry of the table of leaves: a wavefront's

// Leaf of every 64th pair, and of the last one.
__global__ __launch_bounds__(256) void k_pair_leaves(const int64_t *__restrict__ off, int nl,
                                                     int64_t np, int32_t *seg)
{
    const int64_t g = blockIdx.x * (int64_t)256 + threadIdx.x;
    if (g > (np + TP_SEG - 1) / TP_SEG)
        return;
    const int64_t e = min(g * TP_SEG, np - 1);
    int lo = 0, hi = nl - 1;  // last leaf whose pairs start at or before e
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (off[mid] <= e)
            lo = mid;
        else
            hi = mid - 1;
    }
    seg[g] = lo;
}

// Digits and words of the pairs that this lane has of its wavefront's
// TP_ROUNDS rounds of 64 consecutive pairs from e0 (past the end: 0).
template <int BITS, bool FIRST>
__device__ __forceinline__ void tp_load(const PairLists &P, const uint32_t *__restrict__ in,
                                        int64_t e0, uint32_t *dig, uint32_t *word)
{
    const int lane = lane_id();
    if constexpr (FIRST) {
        // the leaves of the rounds' first and last pairs: one leaf or two
        // neighbours nearly always
        int leaf[TP_ROUNDS];
        int64_t start[TP_ROUNDS];
#pragma unroll
        for (int r = 0; r < TP_ROUNDS; ++r) {
            const int64_t g = min(e0 + 64 * r, P.np - 1) / TP_SEG, e = e0 + 64 * r + lane;
            const int lo = P.seg[g], hi = P.seg[g + 1];
            const int64_t s0 = P.off[lo], s1 = P.off[hi];
            leaf[r] = e >= s1 ? hi : lo;
            start[r] = e >= s1 ? s1 : s0;
            if (hi - lo > 1 && e < P.np) {
                int a = lo, b = hi;
                while (a < b) {
                    const int mid = (a + b + 1) >> 1;
                    if (P.off[mid] <= e)
                        a = mid;
                    else
                        b = mid - 1;
                }
                leaf[r] = a;
                start[r] = P.off[a];
            }
        }
        uint32_t target[TP_ROUNDS];
#pragma unroll
        for (int r = 0; r < TP_ROUNDS; ++r) {
            const int64_t e = e0 + 64 * r + lane;
            target[r] = e < P.np ? (uint32_t)P.slots[leaf[r] * P.cap + (e - start[r])] : 0u;
        }
#pragma unroll
        for (int r = 0; r < TP_ROUNDS; ++r) {
            dig[r] = target[r] & ((1u << BITS) - 1u);
            word[r] = ((target[r] >> BITS) << P.leaf_bits) | (uint32_t)leaf[r];
        }
    } else {
        uint32_t p[TP_ROUNDS];
#pragma unroll
        for (int r = 0; r < TP_ROUNDS; ++r) {
            const int64_t e = e0 + 64 * r + lane;
            p[r] = e < P.np ? in[e] : 0u;
        }
#pragma unroll
        for (int r = 0; r < TP_ROUNDS; ++r) {
            dig[r] = p[r] >> P.leaf_bits;
            word[r] = p[r] & ((1u << P.leaf_bits) - 1u);
        }
    }
}

template <int BITS, bool FIRST>
__global__ __launch_bounds__(TP_THREADS) void k_tp_hist(PairLists P,
                                                        const uint32_t *__restrict__ in,
                                                        uint32_t *hist, int nblk)
{
    constexpr int NB = 1 << BITS;
    __shared__ uint32_t h[NB];
    const int t = threadIdx.x;
    for (int i = t; i < NB; i += TP_THREADS)
        h[i] = 0u;
    const int w = __builtin_amdgcn_readfirstlane(t >> 6);
    const int64_t e0 = (int64_t)blockIdx.x * TP_TILE + w * (TP_TILE / TP_WAVES);
    uint32_t dig[TP_ROUNDS], word[TP_ROUNDS];
    tp_load<BITS, FIRST>(P, in, e0, dig, word);
    __syncthreads();
#pragma unroll
    for (int r = 0; r < TP_ROUNDS; ++r)
        if (e0 + 64 * r + lane_id() < P.np)
            atomicAdd(&h[dig[r]], 1u);
    __syncthreads();
    for (int i = t; i < NB; i += TP_THREADS)
        hist[(int64_t)i * nblk + blockIdx.x] = h[i];
}

// Stable scatter of one tile: ranks by ballots per wavefront, the tile in the
// order of its digits in LDS, then each digit's run to its place.  map != null:
// what the words are written as.
template <int BITS, bool FIRST>
__global__ __launch_bounds__(TP_THREADS) void k_tp_scatter(
    PairLists P, const uint32_t *__restrict__ in, const int32_t *__restrict__ map, uint32_t *out,
    const uint32_t *__restrict__ hist, const uint32_t *__restrict__ tot, int nblk)
{
    constexpr int NB = 1 << BITS;
    constexpr int DPT = NB > TP_THREADS ? NB / TP_THREADS : 1;  // digits per thread
    __shared__ uint32_t sword[TP_TILE];
    __shared__ uint16_t sdig[TP_TILE];
    __shared__ uint16_t wrun[TP_WAVES][NB];
    __shared__ uint32_t loff[NB], gofs[NB];
    __shared__ uint32_t wtot[TP_WAVES], wtot2[TP_WAVES];
    const int blk = blockIdx.x, t = threadIdx.x, lane = lane_id();
    const int w = __builtin_amdgcn_readfirstlane(t >> 6);
    for (int i = t; i < TP_WAVES * NB; i += TP_THREADS)
        (&wrun[0][0])[i] = 0;
    const int64_t tile0 = (int64_t)blk * TP_TILE;
    const int nv = (int)min((int64_t)TP_TILE, P.np - tile0);
    const int wbase = w * (TP_TILE / TP_WAVES);
    uint32_t dig[TP_ROUNDS], word[TP_ROUNDS], rank[TP_ROUNDS];
    tp_load<BITS, FIRST>(P, in, tile0 + wbase, dig, word);
    uint32_t gofs_t[DPT], dtot[DPT];
#pragma unroll
    for (int k = 0; k < DPT; ++k) {
        const int d = t * DPT + k;
        gofs_t[k] = d < NB ? hist[(int64_t)d * nblk + blk] : 0u;
        dtot[k] = d < NB ? tot[d] : 0u;
    }
    const uint64_t lt = lanemask_lt();
    __syncthreads();
#pragma unroll
    for (int r = 0; r < TP_ROUNDS; ++r) {
        const bool valid = wbase + r * 64 + lane < nv;
        const uint64_t peers = match_digit<BITS>(dig[r], valid);
        const uint32_t cur = wrun[w][dig[r]];
        rank[r] = cur + (uint32_t)__popcll(peers & lt);
        if (valid && (peers & lt) == 0ull)
            wrun[w][dig[r]] = (uint16_t)(cur + (uint32_t)__popcll(peers));
    }
    __syncthreads();
    // per digit: offsets of the wavefronts, of the digit in the tile, of the
    // tile's run in the output
    uint32_t cnt[DPT], own = 0, own2 = 0;
#pragma unroll
    for (int k = 0; k < DPT; ++k) {
        const int d = t * DPT + k;
        cnt[k] = 0u;
        if (d < NB) {
#pragma unroll
            for (int i = 0; i < TP_WAVES; ++i) {
                const uint32_t c = wrun[i][d];
                wrun[i][d] = (uint16_t)cnt[k];
                cnt[k] += c;
            }
        }
        own += cnt[k];
        own2 += dtot[k];
    }
    uint32_t inc = own, inc2 = own2;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t o = __shfl_up(inc, off), o2 = __shfl_up(inc2, off);
        if (lane >= off) {
            inc += o;
            inc2 += o2;
        }
    }
    if (lane == 63) {
        wtot[w] = inc;
        wtot2[w] = inc2;
    }
    __syncthreads();
    uint32_t lo = inc - own, go = inc2 - own2;
    for (int i = 0; i < w; ++i) {
        lo += wtot[i];
        go += wtot2[i];
    }
#pragma unroll
    for (int k = 0; k < DPT; ++k) {
        const int d = t * DPT + k;
        if (d < NB) {
            loff[d] = lo;
            gofs[d] = go + gofs_t[k] - lo;  // of the digit's run, less its place in the tile
        }
        lo += cnt[k];
        go += dtot[k];
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < TP_ROUNDS; ++r) {
        if (wbase + r * 64 + lane < nv) {
            const uint32_t lp = loff[dig[r]] + wrun[w][dig[r]] + rank[r];
            sword[lp] = word[r];
            sdig[lp] = (uint16_t)dig[r];
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < TP_ROUNDS; ++r) {
        const int j = t + r * TP_THREADS;
        if (j < nv) {
            const uint32_t v = sword[j];
            out[(uint32_t)(gofs[sdig[j]] + (uint32_t)j)] = map ? (uint32_t)map[v] : v;
        }
    }
}

__device__ __forceinline__ uint32_t tp_block_sum(uint32_t v, uint32_t *sh)
{
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1)
        v += __shfl_xor(v, off);
    if (lane_id() == 0)
        sh[threadIdx.x >> 6] = v;
    __syncthreads();
    uint32_t s = 0;
    for (int i = 0; i < (int)(blockDim.x >> 6); ++i)
        s += sh[i];
    __syncthreads();
    return s;
}

// Offsets of the targets from one digit's totals: pairs with a smaller digit.
__global__ __launch_bounds__(256) void k_tp_offsets1(const uint32_t *__restrict__ tot, int nnodes,
                                                     int64_t *off)
{
    __shared__ uint32_t sh[4];
    const int b = blockIdx.x;  // target
    uint32_t v = 0;
    for (int i = threadIdx.x; i < b; i += 256)
        v += tot[i];
    const uint32_t s = tp_block_sum(v, sh);
    if (threadIdx.x == 0)
        off[b] = (int64_t)s;
}

// Offsets of the targets with low digit blockIdx.x.  In the order of the first
// pass the pairs with a smaller low digit end at position p; of high digit h
// come, before target (h, low): the pairs of smaller high digits, those of h in
// the tiles before p's, and those of h in p's tile before p.
template <int BITS>
__global__ __launch_bounds__(256) void k_tp_offsets2(const uint32_t *__restrict__ in,
                                                     int leaf_bits,
                                                     const uint32_t *__restrict__ tot1,
                                                     const uint32_t *__restrict__ hist2,
                                                     const uint32_t *__restrict__ tot2, int nblk,
                                                     int nnodes, int64_t *off)
{
    constexpr int NB = 1 << BITS, PER = NB / 256;
    __shared__ uint32_t cnt[NB];
    __shared__ uint32_t sh[4], sc[4];
    const int low = blockIdx.x, t = threadIdx.x;
    for (int i = t; i < NB; i += 256)
        cnt[i] = 0u;
    uint32_t v = 0;
    for (int i = t; i < low; i += 256)
        v += tot1[i];
    const int64_t p = tp_block_sum(v, sh);
    const int64_t blk = p / TP_TILE;
    for (int64_t e = blk * TP_TILE + t; e < p; e += 256)
        atomicAdd(&cnt[in[e] >> leaf_bits], 1u);
    __syncthreads();
    // digit bases: an exclusive scan, PER consecutive digits per thread
    uint32_t own = 0, dt[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        dt[k] = tot2[t * PER + k];
        own += dt[k];
    }
    uint32_t inc = own;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t x = __shfl_up(inc, o);
        if (lane_id() >= o)
            inc += x;
    }
    if (lane_id() == 63)
        sc[t >> 6] = inc;
    __syncthreads();
    uint32_t base = inc - own;
    for (int i = 0; i < (t >> 6); ++i)
        base += sc[i];
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int h = t * PER + k;
        const int64_t key = ((int64_t)h << BITS) | low;
        if (key <= nnodes)
            off[key] = (int64_t)base + (blk < nblk ? hist2[(int64_t)h * nblk + blk] : dt[k]) +
                       cnt[h];
        base += dt[k];
    }
}

int64_t tp_seg_entries(int64_t np) { return np / TP_SEG + 2; }
int64_t tp_hist_words(int64_t np) { return 1024 * ((np + TP_TILE - 1) / TP_TILE + 1); }

template <int BITS>
static hipError_t transpose_run(const PairLists &P, int key_bits, const int32_t *map, int nnodes,
                                uint32_t *tmp, uint32_t *hist, uint32_t *tot, int64_t *off,
                                uint32_t *out, hipStream_t s)
{
    constexpr int NB = 1 << BITS;
    const int nblk = (int)((P.np + TP_TILE - 1) / TP_TILE);
    uint32_t *tot2 = tot + 1024;
    k_tp_hist<BITS, true><<<nblk, TP_THREADS, 0, s>>>(P, nullptr, hist, nblk);
    hipError_t e = launch_rs_scan(hist, tot, NB, nblk, s);
    if (e != hipSuccess)
        return e;
    if (key_bits <= BITS) {
        k_tp_scatter<BITS, true><<<nblk, TP_THREADS, 0, s>>>(P, nullptr, map, out, hist,
                                                                    tot, nblk);
        k_tp_offsets1<<<nnodes + 1, 256, 0, s>>>(tot, nnodes, off);
        return hipGetLastError();
    }
    k_tp_scatter<BITS, true><<<nblk, TP_THREADS, 0, s>>>(P, nullptr, nullptr, tmp, hist,
                                                                tot, nblk);
    k_tp_hist<BITS, false><<<nblk, TP_THREADS, 0, s>>>(P, tmp, hist, nblk);
    if ((e = launch_rs_scan(hist, tot2, NB, nblk, s)) != hipSuccess)
        return e;
    k_tp_scatter<BITS, false><<<nblk, TP_THREADS, 0, s>>>(P, tmp, map, out, hist, tot2,
                                                                 nblk);
    k_tp_offsets2<BITS><<<NB, 256, 0, s>>>(tmp, P.leaf_bits, tot, hist, tot2, nblk, nnodes,
                                                 off);
    return hipGetLastError();
}

// Width of the digits for targets of key_bits bits; 0: they take more than two
// digits, or the word of the first pass more than 32 bits.
int tp_digit_bits(int key_bits, int leaf_bits)
{
    const int d = key_bits <= 8 ? 8 : key_bits <= 10 ? key_bits : std::max(8, (key_bits + 1) / 2);
    return d <= 10 && std::max(0, key_bits - d) + leaf_bits <= 32 ? d : 0;
}

hipError_t launch_transpose(const PairLists &P, int key_bits, const int32_t *map, int nnodes,
                            int32_t *seg, uint32_t *tmp, uint32_t *hist, uint32_t *tot,
                            int64_t *off, uint32_t *out, hipStream_t s)
{
    const int64_t nseg = (P.np + TP_SEG - 1) / TP_SEG + 1;
    k_pair_leaves<<<(int)((nseg + 255) / 256), 256, 0, s>>>(P.off, P.nl, P.np, seg);
    switch (tp_digit_bits(key_bits, P.leaf_bits)) {
    case 8:
        return transpose_run<8>(P, key_bits, map, nnodes, tmp, hist, tot, off, out, s);
    case 9:
        return transpose_run<9>(P, key_bits, map, nnodes, tmp, hist, tot, off, out, s);
    case 10:
        return transpose_run<10>(P, key_bits, map, nnodes, tmp, hist, tot, off, out, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace fmm
