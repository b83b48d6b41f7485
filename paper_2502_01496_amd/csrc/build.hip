// kd-tree build on gfx950.
//
// The paper's tree (Sec. 2) cuts every cell along its longest axis until a
// cell holds at most a few particles.  The cut used here is the count median
// of the longest axis of the cell's particle bounding box, ties broken by
// (coordinate, Morton rank); both halves keep ascending Morton rank.
//
// Steps (all on the caller's stream):
//   1. global bounding box (ordered-bit atomics, order-free);
//   2. 63-bit Morton keys of positions quantised to 2^21 per axis;
//   3. stable LSD radix sort by key -> Morton rank order (by halves, see
//      sort_by_halves; a tree whose earlier builds met long runs of equal
//      high halves sorts all eight digits instead); few particles are put
//      in the same order by counting (COUNT_SORT_MAX), as in step 4;
//   4. three stable radix sorts by ordered coordinate bits, from rank order,
//      giving per axis the particles sorted by (x_d, rank);
//   5. for cells larger than SUBTREE_MAX, one level at a time: the median of
//      the longest axis is the middle entry of that axis's sorted segment, so
//      the split is a stable partition of the three axis lists; an entry's side
//      follows from comparing its key (coordinate bits, rank) with that of the
//      last left entry;
//   6. every cell of at most SUBTREE_MAX particles is finished by one
//      workgroup in LDS (all levels below it), which writes the final order.
//
// Compiled with -ffp-contract=off: the quantisation and the split-axis test
// are single IEEE operations in the same order as the definition.
#include "fmm_internal.h"

namespace fmm {

// ---------------------------------------------------------------- bbox / keys
__global__ void k_bbox_init(uint64_t *bbox, uint32_t *err)
{
    int t = threadIdx.x;
    if (t < 3) {
        bbox[t] = ~0ull;
        bbox[3 + t] = 0ull;
    }
    if (t == 0)
        err[0] = 0u;
}

__global__ __launch_bounds__(256) void k_bbox(const double *__restrict__ x, int64_t n,
                                              uint64_t *bbox, uint32_t *err)
{
    __shared__ uint64_t sh[4][7];
    uint64_t mn[3] = {~0ull, ~0ull, ~0ull}, mx[3] = {0ull, 0ull, 0ull};
    bool bad = false;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            double v = x[3 * i + d];
            bad |= !isfinite(v);
            uint64_t k = ordbits(v);
            mn[d] = k < mn[d] ? k : mn[d];
            mx[d] = k > mx[d] ? k : mx[d];
        }
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1)
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            uint64_t a = __shfl_xor(mn[d], off);
            uint64_t b = __shfl_xor(mx[d], off);
            mn[d] = a < mn[d] ? a : mn[d];
            mx[d] = b > mx[d] ? b : mx[d];
        }
    const int w = threadIdx.x >> 6;
    uint64_t anybad = __ballot(bad);
    if (lane_id() == 0) {
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            sh[w][d] = mn[d];
            sh[w][3 + d] = mx[d];
        }
        sh[w][6] = anybad ? 1ull : 0ull;
    }
    __syncthreads();
    if (threadIdx.x < 7) {
        const int k = threadIdx.x;
        uint64_t r = sh[0][k];
        for (int i = 1; i < 4; ++i) {
            uint64_t o = sh[i][k];
            r = (k < 3) ? (o < r ? o : r) : (o > r ? o : r);
        }
        if (k < 3)
            atomicMin((unsigned long long *)&bbox[k], (unsigned long long)r);
        else if (k < 6)
            atomicMax((unsigned long long *)&bbox[k], (unsigned long long)r);
        else if (r)
            atomicOr(err, 1u);
    }
}

__device__ __forceinline__ uint64_t spread3(uint64_t v)
{
    v &= 0x1fffffull;
    v = (v | (v << 32)) & 0x1f00000000ffffull;
    v = (v | (v << 16)) & 0x1f0000ff0000ffull;
    v = (v | (v << 8)) & 0x100f00f00f00f00full;
    v = (v | (v << 4)) & 0x10c30c30c30c30c3ull;
    v = (v | (v << 2)) & 0x1249249249249249ull;
    return v;
}

// Grid of the Morton keys from the bounding box (ordered bits).
struct MortonGrid {
    double lo[3], scale;
};

__device__ __forceinline__ MortonGrid morton_grid(const uint64_t *bbox)
{
    MortonGrid g;
    double ext = 0.0;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        g.lo[d] = from_ordbits(bbox[d]);
        double e = from_ordbits(bbox[3 + d]) - g.lo[d];
        if (e > ext)
            ext = e;
    }
    if (ext == 0.0)
        ext = 1.0;
    g.scale = 2097152.0 / ext;
    return g;
}

__device__ __forceinline__ uint64_t morton_key(const double *x, int64_t i, const MortonGrid &g)
{
    uint64_t k = 0;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        double t = floor((x[3 * i + d] - g.lo[d]) * g.scale);
        uint64_t q = t >= 2097151.0 ? 2097151ull : (t >= 0.0 ? (uint64_t)t : 0ull);
        k |= spread3(q) << d;
    }
    return k;
}

__global__ void k_morton(const double *__restrict__ x, int64_t n, const uint64_t *bbox,
                         uint64_t *keys, uint32_t *vals)
{
    const MortonGrid g = morton_grid(bbox);
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        keys[i] = morton_key(x, i, g);
        vals[i] = (uint32_t)i;
    }
}

// Coordinates in Morton-rank order, and the three axis keys (ordered bits,
// value = rank) for the per-axis sorts.
__global__ void k_rank_gather(const double *__restrict__ x, int64_t n, const uint32_t *order,
                              int32_t *r2o, double *xr, uint64_t *keys, uint32_t *vals)
{
    for (int64_t r = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; r < n;
         r += (int64_t)gridDim.x * blockDim.x) {
        int64_t i = order[r];
        r2o[r] = (int32_t)i;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            double v = x[3 * i + d];
            xr[d * n + r] = v;
            keys[d * n + r] = ordbits(v);
            vals[d * n + r] = (uint32_t)r;
        }
    }
}

// ---------------------------------------------------------------- few particles
// Up to COUNT_SORT_MAX particles the order is found by counting: the place of
// a key is the number of keys before it, in (key, position) order.  The radix
// sorts take some 15 launches each for one or two tiles, bound by the launches
// and by the one or two workgroups of a launch; counting is n^2 comparisons
// of two instructions over all CUs in one launch.  A whole build takes 45 us
// (n = 1000), 87 (4096), 124 (8192) and 165 (12288) instead of 134, 178, 194
// and 182 with the radix sorts; at 16384 it would be 219 against 189.
constexpr int COUNT_SORT_MAX = 12288;
constexpr int CR_THREADS = 1024, CR_WAVES = CR_THREADS / 64;

// Bounding box (with the non-finite check) and Morton keys by one workgroup;
// clears the counters of long runs that a radix sort would set.
__global__ __launch_bounds__(CR_THREADS) void k_morton_few(const double *__restrict__ x, int n,
                                                           uint64_t *bbox, uint64_t *keys,
                                                           uint32_t *run_cnt, uint32_t *err)
{
    __shared__ uint64_t sh[CR_WAVES][7];
    __shared__ uint64_t box[6];
    const int t = threadIdx.x, w = t >> 6;
    uint64_t mn[3] = {~0ull, ~0ull, ~0ull}, mx[3] = {0ull, 0ull, 0ull};
    bool bad = false;
    for (int i = t; i < n; i += CR_THREADS)
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            const double v = x[3 * i + d];
            bad |= !isfinite(v);
            const uint64_t k = ordbits(v);
            mn[d] = k < mn[d] ? k : mn[d];
            mx[d] = k > mx[d] ? k : mx[d];
        }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1)
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            const uint64_t a = __shfl_xor(mn[d], off), b = __shfl_xor(mx[d], off);
            mn[d] = a < mn[d] ? a : mn[d];
            mx[d] = b > mx[d] ? b : mx[d];
        }
    const uint64_t anybad = __ballot(bad);
    if (lane_id() == 0) {
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            sh[w][d] = mn[d];
            sh[w][3 + d] = mx[d];
        }
        sh[w][6] = anybad ? 1ull : 0ull;
    }
    __syncthreads();
    if (t < 7) {
        uint64_t r = sh[0][t];
        for (int i = 1; i < CR_WAVES; ++i) {
            const uint64_t o = sh[i][t];
            r = t < 3 ? (o < r ? o : r) : (o > r ? o : r);
        }
        if (t < 6) {
            box[t] = r;
            bbox[t] = r;
        } else {
            err[0] = (uint32_t)r;
        }
    }
    if (t < 2)
        run_cnt[t] = 0u;
    __syncthreads();
    const MortonGrid g = morton_grid(box);
    for (int i = t; i < n; i += CR_THREADS)
        keys[i] = morton_key(x, i, g);
}

// Place of element blockIdx.x * 64 + lane among the n keys in (key, position)
// order: each wavefront counts over its share of the keys (read as scalars),
// the shares are added in LDS.  Valid in the first wavefront.
__device__ __forceinline__ int count_rank(const uint64_t *__restrict__ keys, int n, uint64_t ke)
{
    __shared__ int part[CR_WAVES][64];
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = lane_id();
    const int i0 = blockIdx.x * 64, e = i0 + lane;
    const int per = (n + CR_WAVES - 1) / CR_WAVES;
    const int lo = min(n, w * per), hi = min(n, lo + per);
    // keys of earlier positions, of this wavefront's own, of later ones
    const int a = min(max(i0, lo), hi), b = min(max(i0 + 64, lo), hi);
    int cnt = 0;
#pragma unroll 8
    for (int j = lo; j < a; ++j)
        cnt += keys[j] <= ke ? 1 : 0;
    for (int j = a; j < b; ++j)
        cnt += keys[j] < ke || (keys[j] == ke && j < e) ? 1 : 0;
#pragma unroll 8
    for (int j = b; j < hi; ++j)
        cnt += keys[j] < ke ? 1 : 0;
    part[w][lane] = cnt;
    __syncthreads();
    int r = 0;
    if (w == 0)
        for (int i = 0; i < CR_WAVES; ++i)
            r += part[i][lane];
    return r;
}

// Morton order; xr != null: also what k_rank_gather makes of it.
__global__ __launch_bounds__(CR_THREADS) void k_rank_morton(
    const uint64_t *__restrict__ keys, const double *__restrict__ x, int n, uint32_t *order,
    int32_t *r2o, double *xr, uint64_t *akeys)
{
    const int e = blockIdx.x * 64 + lane_id();
    const int r = count_rank(keys, n, keys[min(e, n - 1)]);
    if (threadIdx.x >= 64 || e >= n)
        return;
    order[r] = (uint32_t)e;
    if (!xr)
        return;
    r2o[r] = e;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const double v = x[3 * e + d];
        xr[d * (int64_t)n + r] = v;
        akeys[d * (int64_t)n + r] = ordbits(v);
    }
}

// Axis lists: the ranks in (coordinate, rank) order, axis blockIdx.y.
__global__ __launch_bounds__(CR_THREADS) void k_rank_axes(const uint64_t *__restrict__ akeys, int n,
                                                          uint32_t *lists)
{
    const uint64_t *k = akeys + (int64_t)blockIdx.y * n;
    const int e = blockIdx.x * 64 + lane_id();
    const int r = count_rank(k, n, k[min(e, n - 1)]);
    if (threadIdx.x < 64 && e < n)
        lists[(int64_t)blockIdx.y * n + r] = (uint32_t)e;
}

// ---------------------------------------------------------------- radix sort
// Stable LSD radix sort of B independent (key u64, value u32) arrays of
// length n laid out back to back.  Per 8-bit pass: per-tile digit histograms,
// a scan per (digit, array) over the tiles that also stores the digit's
// total, then a stable scatter that adds the digit bases (a scan of the 256
// totals in LDS, so no tile updates a shared counter).  Inside a tile the 16
// waves take consecutive sixteenths; a wave ranks its 64 keys of a round with
// ballot-based digit matching, so rank order = input order.
__global__ void k_rs_zero(uint32_t *p, int64_t cnt)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < cnt;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = 0u;
}

template <typename K, int BITS>
__global__ __launch_bounds__(RS_THREADS) void k_rs_hist(const K *__restrict__ keys, int64_t n,
                                                        int shift, uint32_t *hist, int nblk)
{
    constexpr int NB = 1 << BITS;  // digits (at most RS_THREADS)
    __shared__ uint32_t h[NB];
    int b = blockIdx.y, blk = blockIdx.x, t = threadIdx.x;
    if (t < NB)
        h[t] = 0u;
    __syncthreads();
    const K *k = keys + (int64_t)b * n;
    int64_t base = (int64_t)blk * RS_TILE;
    // all loads first (indices past the end re-read key n - 1, not counted)
    K kr[RS_ROUNDS];
#pragma unroll
    for (int r = 0; r < RS_ROUNDS; ++r)
        kr[r] = k[min(base + r * RS_THREADS + t, n - 1)];
#pragma unroll
    for (int r = 0; r < RS_ROUNDS; ++r)
        if (base + r * RS_THREADS + t < n)
            atomicAdd(&h[(uint32_t)(kr[r] >> shift) & (NB - 1u)], 1u);
    __syncthreads();
    if (t < NB)
        hist[((int64_t)b * NB + t) * nblk + blk] = h[t];
}

// Exclusive scan across one block of up to 256 threads (values <= 2^32).
__device__ __forceinline__ uint32_t block_excl_scan_u32(uint32_t v, uint32_t *sh, uint32_t &total)
{
    int t = threadIdx.x, lane = lane_id(), w = t >> 6, nw = blockDim.x >> 6;
    uint32_t inc = v;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        uint32_t o = __shfl_up(inc, off);
        if (lane >= off)
            inc += o;
    }
    if (lane == 63)
        sh[w] = inc;
    __syncthreads();
    uint32_t wbase = 0, tot = 0;
    for (int i = 0; i < nw; ++i) {
        uint32_t s = sh[i];
        wbase += i < w ? s : 0u;
        tot += s;
    }
    __syncthreads();
    total = tot;
    return wbase + inc - v;
}

// Row (digit d of array b) of the tile histograms -> offsets of the tiles
// within the digit's output run; the row total goes to tot.  A row is one chain
// of block scans, so a lane takes RS_SCAN_PER tiles of a scan (5100 tiles, the far
// pairs of the binary, 2^19 particles: 19.7 us with one tile per lane; the scans
// of a pass over Plummer's reverse pass, 2^19, 25.7 -> 17.7 us on average).
constexpr int RS_SCAN_PER = 8;
__global__ __launch_bounds__(RS_SCAN_THREADS) void k_rs_scan(uint32_t *hist, uint32_t *tot,
                                                             int nblk)
{
    __shared__ uint32_t sh[8];
    const int nb = gridDim.x;  // digits
    int d = blockIdx.x, b = blockIdx.y, t = threadIdx.x;
    uint32_t *row = hist + ((int64_t)b * nb + d) * nblk;
    uint32_t run = 0;
    for (int c0 = 0; c0 < nblk; c0 += RS_SCAN_THREADS * RS_SCAN_PER) {
        const int i0 = c0 + t * RS_SCAN_PER;
        uint32_t v[RS_SCAN_PER], sum = 0;
#pragma unroll
        for (int k = 0; k < RS_SCAN_PER; ++k)
            v[k] = i0 + k < nblk ? row[i0 + k] : 0u;
#pragma unroll
        for (int k = 0; k < RS_SCAN_PER; ++k)
            sum += v[k];
        uint32_t total;
        uint32_t ex = run + block_excl_scan_u32(sum, sh, total);
#pragma unroll
        for (int k = 0; k < RS_SCAN_PER; ++k) {
            if (i0 + k < nblk)
                row[i0 + k] = ex;
            ex += v[k];
        }
        run += total;
    }
    if (t == 0)
        tot[b * nb + d] = run;
}

hipError_t launch_rs_scan(uint32_t *hist, uint32_t *tot, int digits, int nblk, hipStream_t s)
{
    k_rs_scan<<<dim3(digits, 1), RS_SCAN_THREADS, 0, s>>>(hist, tot, nblk);
    return hipGetLastError();
}

// Stable scatter of one tile: rank the keys by digit (per wave, ballot
// matching; waves in order), place the tile digit-sorted in LDS, then write
// each digit's run to its global position with consecutive threads on
// consecutive addresses.  VALS = false: keys only (no values loaded, staged
// in LDS or written).
// FOLD: hist holds the counts of the tiles as they are (few tiles), and every
// tile sums the rows itself.
template <typename K, int BITS, bool VALS, bool FOLD>
__global__ __launch_bounds__(RS_THREADS) void k_rs_scatter(
    const K *__restrict__ kin, const uint32_t *__restrict__ vin, K *kout, uint32_t *vout,
    int64_t n, int shift, const uint32_t *__restrict__ hist, const uint32_t *__restrict__ tot,
    int nblk)
{
    constexpr int NB = 1 << BITS;  // digits, one per thread of the first NB threads
    constexpr uint32_t DM = NB - 1u;
    __shared__ K skey[RS_TILE];
    __shared__ uint32_t sval[VALS ? RS_TILE : 1];
    __shared__ uint16_t wrun[RS_WAVES][NB];
    __shared__ uint32_t loff[NB];
    __shared__ uint32_t gofs[NB];
    __shared__ uint32_t wtot[NB / 64], wtot2[NB / 64];
    const int b = blockIdx.y, blk = blockIdx.x, t = threadIdx.x, w = t >> 6, lane = lane_id();
    for (int i = t; i < RS_WAVES * NB; i += RS_THREADS)
        (&wrun[0][0])[i] = 0;
    __syncthreads();
    const K *k = kin + (int64_t)b * n;
    const uint32_t *v = VALS ? vin + (int64_t)b * n : nullptr;
    const int64_t tile0 = (int64_t)blk * RS_TILE;
    const int nv = (int)min((int64_t)RS_TILE, n - tile0);
    const int wbase = w * (RS_TILE / RS_WAVES);
    K key[RS_ROUNDS];
    uint32_t val[RS_ROUNDS];
    uint32_t rank[RS_ROUNDS];
    const uint64_t lt = lanemask_lt();
#pragma unroll
    for (int r = 0; r < RS_ROUNDS; ++r) {
        const int i = wbase + r * 64 + lane;
        key[r] = i < nv ? k[tile0 + i] : K(0);
        val[r] = (VALS && i < nv) ? v[tile0 + i] : 0u;
    }
    // this tile's offsets within the digit runs and the digit totals, loaded
    // while the keys are in flight
    uint32_t gofs_t = 0u, dtot = 0u;
    if (t < NB) {
        const uint32_t *row = hist + ((int64_t)b * NB + t) * nblk;
        if constexpr (FOLD) {
#pragma unroll 8
            for (int i = 0; i < nblk; ++i) {
                const uint32_t c = row[i];
                gofs_t += i < blk ? c : 0u;
                dtot += c;
            }
        } else {
            gofs_t = row[blk];
            dtot = tot[b * NB + t];
        }
    }
#pragma unroll
    for (int r = 0; r < RS_ROUNDS; ++r) {
        const bool valid = wbase + r * 64 + lane < nv;
        const uint32_t d = valid ? (uint32_t)(key[r] >> shift) & DM : 0u;
        const uint64_t peers = match_digit<BITS>(d, valid);
        const uint32_t cur = wrun[w][d];
        rank[r] = cur + (uint32_t)__popcll(peers & lt);
        if (valid && (peers & lt) == 0ull)
            wrun[w][d] = (uint16_t)(cur + (uint32_t)__popcll(peers));
    }
    __syncthreads();
    // per digit: offsets of the waves, then the tile-local digit offsets
    uint32_t cnt = 0;
    if (t < NB) {
#pragma unroll
        for (int i = 0; i < RS_WAVES; ++i) {
            const uint32_t c = wrun[i][t];
            wrun[i][t] = (uint16_t)cnt;
            cnt += c;
        }
        // exclusive scans over the digits: tile-local offsets (of cnt) and
        // the digit bases (of the totals)
        uint32_t inc = cnt, inc2 = dtot;
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
        loff[t] = inc - cnt;
        gofs[t] = gofs_t + (inc2 - dtot);
    }
    __syncthreads();
    if (t < NB) {
        uint32_t add = 0, add2 = 0;
        for (int i = 0; i < w; ++i) {
            add += wtot[i];
            add2 += wtot2[i];
        }
        loff[t] += add;
        gofs[t] += add2;
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < RS_ROUNDS; ++r) {
        if (wbase + r * 64 + lane < nv) {
            const uint32_t d = (uint32_t)(key[r] >> shift) & DM;
            const uint32_t lp = loff[d] + wrun[w][d] + rank[r];
            skey[lp] = key[r];
            if constexpr (VALS)
                sval[lp] = val[r];
        }
    }
    __syncthreads();
    K *ko = kout + (int64_t)b * n;
    uint32_t *vo = VALS ? vout + (int64_t)b * n : nullptr;
    for (int j = t; j < nv; j += RS_THREADS) {
        const K kk = skey[j];
        const uint32_t d = (uint32_t)(kk >> shift) & DM;
        const int64_t gp = (int64_t)gofs[d] + (j - (int)loff[d]);
        ko[gp] = kk;
        if constexpr (VALS)
            vo[gp] = sval[j];
    }
}

// Up to this many tiles a pass has no scan launch: its tiles sum the rows of the
// counts themselves.  The build (eight passes) of 30011 particles (8 tiles) takes
// 208 instead of 231 us, of 131072 (32) 244 instead of 270, of 262144 (64) 294
// instead of 310, of 300000 326 instead of 337; of 400000 376 either way, of
// 524288 (128) it would be 411 against 402.
constexpr int RS_FOLD_TILES = 64;

// One pass: counts, scan, scatter (vin == nullptr: keys only).
template <typename K, int BITS>
static void radix_pass(const K *kin, const uint32_t *vin, K *kout, uint32_t *vout, int64_t n, int B,
                       int shift, uint32_t *hist, uint32_t *tot, hipStream_t s)
{
    constexpr int NB = 1 << BITS;
    const int nblk = (int)((n + RS_TILE - 1) / RS_TILE);
    const bool fold = nblk <= RS_FOLD_TILES;
    const dim3 g(nblk, B);
    k_rs_hist<K, BITS><<<g, RS_THREADS, 0, s>>>(kin, n, shift, hist, nblk);
    if (!fold)
        k_rs_scan<<<dim3(NB, B), RS_SCAN_THREADS, 0, s>>>(hist, tot, nblk);
    auto run = [&](auto kernel) {
        kernel<<<g, RS_THREADS, 0, s>>>(kin, vin, kout, vout, n, shift, hist, tot, nblk);
    };
    if (vin && fold)
        run(k_rs_scatter<K, BITS, true, true>);
    else if (vin)
        run(k_rs_scatter<K, BITS, true, false>);
    else if (fold)
        run(k_rs_scatter<K, BITS, false, true>);
    else
        run(k_rs_scatter<K, BITS, false, false>);
}

// Sort B arrays of n (key, value) pairs by the low BITS * passes key bits
// (v0 == v1 == nullptr: keys only), BITS = 8 or 10 bits per pass.  The result
// ends in (k0, v0) after an even number of passes, in (k1, v1) after an odd
// one.  hist needs B * 2^BITS * ceil(n / RS_TILE) words, tot
// passes * B * 2^BITS.
template <typename K, int BITS>
static hipError_t radix_sort(K *k0, uint32_t *v0, K *k1, uint32_t *v1, int64_t n, int B,
                             int passes, uint32_t *hist, uint32_t *tot, hipStream_t s)
{
    constexpr int NB = 1 << BITS;
    int nblk = (int)((n + RS_TILE - 1) / RS_TILE);
    if (nblk == 0)
        return hipSuccess;
    for (int pass = 0; pass < passes; ++pass) {
        int shift = BITS * pass;
        K *ki = (pass & 1) ? k1 : k0, *ko = (pass & 1) ? k0 : k1;
        uint32_t *vi = (pass & 1) ? v1 : v0, *vo = (pass & 1) ? v0 : v1;
        uint32_t *tp = tot + (int64_t)pass * B * NB;
        radix_pass<K, BITS>(ki, vi, ko, vo, n, B, shift, hist, tp, s);
    }
    return hipGetLastError();
}

hipError_t radix_sort_u64(uint64_t *k0, uint32_t *v0, uint64_t *k1, uint32_t *v1, int64_t n,
                          int B, int passes, uint32_t *hist, uint32_t *tot, hipStream_t s,
                          int digit_bits)
{
    return digit_bits == 10
               ? radix_sort<uint64_t, 10>(k0, v0, k1, v1, n, B, passes, hist, tot, s)
               : radix_sort<uint64_t, 8>(k0, v0, k1, v1, n, B, passes, hist, tot, s);
}

// 32-bit keys: half the key traffic of the 64-bit sort.
hipError_t radix_sort_u32(uint32_t *k0, uint32_t *v0, uint32_t *k1, uint32_t *v1, int64_t n,
                          int B, int passes, uint32_t *hist, uint32_t *tot, hipStream_t s,
                          int digit_bits)
{
    return digit_bits == 10
               ? radix_sort<uint32_t, 10>(k0, v0, k1, v1, n, B, passes, hist, tot, s)
               : radix_sort<uint32_t, 8>(k0, v0, k1, v1, n, B, passes, hist, tot, s);
}

// Passes and digit width for keys of `bits` bits: 10-bit digits where they
// take fewer passes than 8-bit ones.
void radix_plan(int bits, int &passes, int &digit_bits)
{
    const int p8 = (bits + 7) / 8, p10 = (bits + 9) / 10;
    digit_bits = p10 < p8 ? 10 : 8;
    passes = p10 < p8 ? p10 : p8;
}

// ---------------------------------------------------------------- (key, value) by halves
// Order by (key, value), the values being the input positions (so this is a
// stable sort by key): four LSD passes over the high 32 key bits, then the
// runs of equal high halves are put in (low half, value) order.  Runs of at
// most RUN_SHORT entries are ranked by one thread per entry; the (rare)
// longer ones by one workgroup each.  For the sorts of the build (Morton keys
// and ordered coordinate bits of spread-out particles) nearly every run has
// one entry, so this replaces the four low passes by one light pass.
constexpr int RUN_SHORT = 64;

__device__ __forceinline__ uint32_t hi32(uint64_t k) { return (uint32_t)(k >> 32); }

// A block stages its 256 entries with RUN_SHORT + 1 more on each side in
// LDS (coalesced loads).  The entries that begin a run are the set bits of one
// word per 64 entries, so a run's ends are found in two words each way, and
// only the ranks inside it are counted entry by entry.  Against walking along the
// runs in LDS, per sort: 437 -> 229 us (binary, 2^24 particles), 75 -> 52 us
// (clumpy cube, 2^22), 10.4 -> 8.9 us (binary, 2^19).
constexpr int RUN_BLOCK = 256;
constexpr int RUN_HALO = RUN_SHORT + 1;
constexpr int RUN_WIN = RUN_BLOCK + 2 * RUN_HALO;
static_assert(RUN_SHORT <= 64, "a run lies within two words of its entries");

__global__ __launch_bounds__(RUN_BLOCK) void k_run_fix(const uint64_t *__restrict__ kin,
                                                       const uint32_t *__restrict__ vin,
                                                       uint32_t *vout, int64_t n,
                                                       uint32_t *long_cnt, int64_t *long_list,
                                                       int64_t long_cap, uint32_t *err)
{
    __shared__ uint32_t shi[RUN_WIN], slo[RUN_WIN], sv[RUN_WIN];
    __shared__ uint64_t head[(RUN_WIN + 63) / 64];
    const int b = blockIdx.y, t = threadIdx.x;
    const uint64_t *k = kin + (int64_t)b * n;
    const uint32_t *v = vin + (int64_t)b * n;
    uint32_t *vo = vout + (int64_t)b * n;
    for (int64_t base = (int64_t)blockIdx.x * RUN_BLOCK; base < n;
         base += (int64_t)gridDim.x * RUN_BLOCK) {
        // window [base - RUN_HALO, base + RUN_BLOCK + RUN_HALO) of the array
        for (int i = t; i < RUN_WIN; i += RUN_BLOCK) {
            const int64_t g = base - RUN_HALO + i;
            if (g >= 0 && g < n) {
                const uint64_t kg = k[g];
                shi[i] = hi32(kg);
                slo[i] = (uint32_t)kg;
                sv[i] = v[g];
            }
        }
        __syncthreads();
        // a run begins where the high half changes, at the array's first entry
        // and past its last (the window's first entry decides no run of at
        // most RUN_SHORT entries)
        for (int i = t; (i & ~63) < RUN_WIN; i += RUN_BLOCK) {
            const int64_t g = base - RUN_HALO + i;
            const bool hd = i < RUN_WIN && (g == 0 || g >= n || (g > 0 && i > 0 &&
                                                                 shi[i] != shi[i - 1]));
            const uint64_t w = __ballot(hd);
            if ((i & 63) == 0)
                head[i >> 6] = w;
        }
        __syncthreads();
        const int64_t p = base + t;
        if (p < n) {
            const int i = t + RUN_HALO;  // window index of p
            const int w = i >> 6, sh = i & 63;
            const uint64_t hw = head[w];
            const uint64_t at = hw & (~0ull >> (63 - sh)), after = hw & (~0ull << sh << 1);
            const uint64_t before = head[w - 1], next = head[w + 1];  // 1 <= w, w + 1 <= 6
            const uint32_t vp = sv[i];
            const bool prev_same = !((hw >> sh) & 1);
            // the run [ia, ie)
            const int ia = at ? 64 * w + 63 - __clzll(at) : 64 * w - 1 - __clzll(before);
            const int ie = after ? 64 * w + __builtin_ctzll(after)
                                 : 64 * (w + 1) + (next ? __builtin_ctzll(next) : 0);
            const bool lng = !(at | before) || !(after | next) || ie - ia > RUN_SHORT;
            if (!lng && ie - ia == 1) {
                // a run of one entry (nearly all of them)
                vo[p] = vp;
            } else {
                if (lng) {
                    if (!prev_same) {
                        const uint32_t slot = atomicAdd(long_cnt, 1u);
                        if ((int64_t)slot < long_cap)
                            long_list[slot] = ((int64_t)b << 40) | p;
                        else
                            atomicOr(err, 8u);
                    }
                } else {
                    const uint32_t lp = slo[i];
                    int r = 0;
                    for (int q = ia; q < ie; ++q) {
                        const uint32_t lq = slo[q], vq = sv[q];
                        r += (lq < lp || (lq == lp && vq < vp)) ? 1 : 0;
                    }
                    vo[p - (i - ia) + r] = vp;
                }
            }
        }
        __syncthreads();
    }
}

// One workgroup per long run: find its end, then a stable LSD radix sort of
// the low key half in four 8-bit passes, ping-ponging between the run's
// segments of the input and output arrays.  The values of a run are already
// ascending (the high-half passes are stable and the values are the input
// positions), so the stable sort by the low half leaves it in (low half,
// value) order.
__global__ __launch_bounds__(RS_THREADS) void k_run_long(uint64_t *kin, uint32_t *vin,
                                                         uint64_t *kout, uint32_t *vout, int64_t n,
                                                         uint32_t *long_cnt,
                                                         const int64_t *__restrict__ long_list,
                                                         int64_t long_cap)
{
    __shared__ uint32_t hist[256];
    __shared__ uint32_t base[256];
    __shared__ uint32_t wcnt[RS_WAVES][256];
    __shared__ uint32_t ctot[256];
    __shared__ int64_t end_sh;
    const int t = threadIdx.x, w = t >> 6, lane = lane_id();
    const uint64_t lt = lanemask_lt();
    const int64_t nl = min((int64_t)*long_cnt, long_cap);
    for (int64_t r = blockIdx.x; r < nl; r += gridDim.x) {
        const int64_t code = long_list[r];
        const int b = (int)(code >> 40);
        const int64_t a = code & ((1ll << 40) - 1);
        uint64_t *K[2] = {kin + (int64_t)b * n, kout + (int64_t)b * n};
        uint32_t *V[2] = {vin + (int64_t)b * n, vout + (int64_t)b * n};
        const uint32_t hp = hi32(K[0][a]);
        // end of the run: first position with another high half (or n)
        if (t == 0)
            end_sh = n;
        __syncthreads();
        for (int64_t c0 = a; c0 < n; c0 += RS_THREADS) {
            const int64_t q = c0 + t;
            if (q < n && hi32(K[0][q]) != hp)
                atomicMin((unsigned long long *)&end_sh, (unsigned long long)q);
            __syncthreads();
            const bool found = end_sh < n;
            __syncthreads();
            if (found)
                break;
        }
        const int64_t L = end_sh - a;
        if (t == 0)
            atomicAdd(&long_cnt[1], (uint32_t)L);  // entries in long runs, for the host
        for (int pass = 0; pass < 4; ++pass) {
            const int src = pass & 1, dst = src ^ 1;
            const uint64_t *ks = K[src] + a;
            const uint32_t *vs = V[src] + a;
            uint64_t *kd = K[dst] + a;
            uint32_t *vd = V[dst] + a;
            const int sh = 8 * pass;
            auto digit = [&](int64_t i) -> uint32_t { return ((uint32_t)ks[i] >> sh) & 255u; };
            if (t < 256)
                hist[t] = 0u;
            __syncthreads();
            for (int64_t i = t; i < L; i += RS_THREADS)
                atomicAdd(&hist[digit(i)], 1u);
            __syncthreads();
            if (t == 0) {
                uint32_t run = 0;
                for (int d = 0; d < 256; ++d) {
                    base[d] = run;
                    run += hist[d];
                }
            }
            __syncthreads();
            for (int64_t c0 = 0; c0 < L; c0 += RS_THREADS) {
                const int64_t i = c0 + t;
                const bool valid = i < L;
                const uint32_t d = valid ? digit(i) : 0u;
                for (int j = t; j < RS_WAVES * 256; j += RS_THREADS)
                    (&wcnt[0][0])[j] = 0u;
                __syncthreads();
                const uint64_t peers = match_digit<8>(d, valid);
                const uint32_t rk = (uint32_t)__popcll(peers & lt);
                if (valid && (peers & lt) == 0ull)
                    wcnt[w][d] = (uint32_t)__popcll(peers);
                __syncthreads();
                if (t < 256) {
                    uint32_t run = 0;
                    for (int ww = 0; ww < RS_WAVES; ++ww) {
                        const uint32_t c = wcnt[ww][t];
                        wcnt[ww][t] = run;
                        run += c;
                    }
                    ctot[t] = run;
                }
                __syncthreads();
                if (valid) {
                    const int64_t pos = (int64_t)base[d] + wcnt[w][d] + rk;
                    kd[pos] = ks[i];
                    vd[pos] = vs[i];
                }
                __syncthreads();
                if (t < 256)
                    base[t] += ctot[t];
                __syncthreads();
            }
        }
        // four passes end in the input arrays: copy the run to the output
        for (int64_t i = t; i < L; i += RS_THREADS)
            V[1][a + i] = V[0][a + i];
        __syncthreads();
    }
}

// Sort B arrays of (key, position) pairs held in (k0, v0); the sorted positions
// land in vout, (k1, v1) is work space.  long_list: B * (n / (RUN_SHORT + 1) + 1)
// entries; long_cnt[0] counts the long runs, long_cnt[1] their entries.
hipError_t sort_by_halves(uint64_t *k0, uint32_t *v0, uint64_t *k1, uint32_t *v1, uint32_t *vout,
                          int64_t n, int B, uint32_t *hist, uint32_t *tot, uint32_t *long_cnt,
                          int64_t *long_list, uint32_t *err, hipStream_t s)
{
    const int nblk = (int)((n + RS_TILE - 1) / RS_TILE);
    if (nblk == 0)
        return hipSuccess;
    const int64_t long_cap = (int64_t)B * (n / (RUN_SHORT + 1) + 1);
    k_rs_zero<<<1, 64, 0, s>>>(long_cnt, 2);
    for (int pass = 0; pass < 4; ++pass) {
        const int shift = 32 + 8 * pass;
        uint64_t *ki = (pass & 1) ? k1 : k0, *ko = (pass & 1) ? k0 : k1;
        uint32_t *vi = (pass & 1) ? v1 : v0, *vo = (pass & 1) ? v0 : v1;
        uint32_t *tp = tot + (int64_t)pass * B * 256;
        radix_pass<uint64_t, 8>(ki, vi, ko, vo, n, B, shift, hist, tp, s);
    }
    const int gf = (int)std::min<int64_t>((n + 255) / 256, 4096);
    k_run_fix<<<dim3(gf, B), 256, 0, s>>>(k0, v0, vout, n, long_cnt, long_list, long_cap, err);
    k_run_long<<<256, RS_THREADS, 0, s>>>(k0, v0, k1, vout, n, long_cnt, long_list, long_cap);
    return hipGetLastError();
}

// ---------------------------------------------------------------- level kernels
// Longest axis of a node from its three sorted lists (first = min, last = max).
__device__ __forceinline__ int node_axis(const uint32_t *L, int64_t n, const double *xr,
                                         int64_t f, int64_t c)
{
    int ax = 0;
    double best = 0.0;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        double lo = xr[d * n + L[d * n + f]];
        double hi = xr[d * n + L[d * n + f + c - 1]];
        double e = hi - lo;
        if (d == 0 || e > best) {
            best = e;
            ax = d;
        }
    }
    return ax;
}

// The split of a cell: the left child takes the first ceil(c/2) entries of
// the longest axis's list, i.e. the particles whose key (ordered coordinate
// bits, Morton rank) is at most the key of entry ceil(c/2) - 1.
struct Split {
    int64_t f, nl;
    int ax;
    uint64_t ob;  // ordered coordinate bits of the last left entry
    uint32_t rm;  // its Morton rank
};

__device__ __forceinline__ Split node_split(const uint32_t *L, int64_t n, const double *xr,
                                            int64_t f, int64_t c)
{
    Split S;
    S.f = f;
    S.nl = (c + 1) / 2;
    S.ax = node_axis(L, n, xr, f, c);
    S.rm = L[S.ax * n + f + S.nl - 1];
    S.ob = ordbits(xr[S.ax * n + S.rm]);
    return S;
}

// Sides of a chunk of one list (also stored per position for the scatter)
// and the chunk's left count.  A chunk holds at most LVL_CHUNK entries, PER
// per thread: the entries are loaded before the split is found and the
// coordinates gathered all at once, so a thread waits for two memory round
// trips rather than two per entry.
__global__ __launch_bounds__(LVL_THREADS) void k_lvl_count(
    const uint32_t *__restrict__ L, int64_t n, const double *__restrict__ xr,
    const int32_t *blk_node, const int32_t *blk_start, const int32_t *blk_end,
    const int32_t *first, const int32_t *count, int32_t *axis_out, uint8_t *side, int32_t *cnt,
    int stride)
{
    constexpr int PER = LVL_CHUNK / LVL_THREADS;
    __shared__ uint32_t sh[8];
    const int b = blockIdx.x, d = blockIdx.y, t = threadIdx.x;
    const int v = blk_node[b];
    const int64_t s0 = blk_start[b], e0 = blk_end[b];
    const uint32_t *Ld = L + d * n;
    // loads past the chunk's end re-read its last entry (a chunk is never
    // empty) and are discarded, so that every load is issued unconditionally
    uint32_t r[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k)
        r[k] = Ld[min(s0 + t + k * LVL_THREADS, e0 - 1)];
    const Split S = node_split(L, n, xr, first[v], count[v]);
    if (d == 0 && t == 0 && s0 == S.f)
        axis_out[v] = S.ax;
    uint32_t g[PER];
    if (d == S.ax) {
#pragma unroll
        for (int k = 0; k < PER; ++k)
            g[k] = s0 + t + k * LVL_THREADS - S.f < S.nl ? 1u : 0u;
    } else {
        uint64_t o[PER];
#pragma unroll
        for (int k = 0; k < PER; ++k)
            o[k] = ordbits(xr[S.ax * n + r[k]]);
#pragma unroll
        for (int k = 0; k < PER; ++k)
            g[k] = (o[k] < S.ob || (o[k] == S.ob && r[k] <= S.rm)) ? 1u : 0u;
    }
    uint8_t *sd = side + d * n;
    uint32_t c = 0;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int64_t p = s0 + t + k * LVL_THREADS;
        if (p < e0) {
            sd[p] = (uint8_t)g[k];
            c += g[k];
        }
    }
    uint32_t total;
    block_excl_scan_u32(c, sh, total);
    if (t == 0)
        cnt[d * stride + b] = (int32_t)total;
}

// Sides by Morton rank at one level: each cell's longest-axis list gives
// them by position (its first ceil(c/2) entries go left), and the other
// lists of the cell then look their entries' sides up by rank (one byte per
// particle instead of a gathered coordinate).  For trees of LVL_BYRANK_MIN
// particles or more, whose coordinate arrays miss in L2; smaller ones gather
// the coordinates and save the extra launch per level.
constexpr int64_t LVL_BYRANK_MIN = int64_t(1) << 20;
// Above LVL_BITS_ABOVE particles the lookups read a bit per particle, packed by
// k_side_bits: the bytes then come near an XCD's L2 (4 MiB) and the lookups miss
// it, the bits fit up to 2^25 particles.  Over the levels of a build, lookups and
// packing: 1402 -> 1044 + 65 us (2^24 particles), 280 -> 190 + 55 us (2^22); at
// 2^21 the 5 us of packing a level are as much as they save.
constexpr int64_t LVL_BITS_ABOVE = int64_t(1) << 21;
__global__ __launch_bounds__(LVL_THREADS) void k_lvl_side(
    const uint32_t *__restrict__ L, int64_t n, const double *__restrict__ xr,
    const int32_t *blk_node, const int32_t *blk_start, const int32_t *blk_end,
    const int32_t *first, const int32_t *count, int32_t *axis_out, uint8_t *byrank)
{
    constexpr int PER = LVL_CHUNK / LVL_THREADS;
    const int b = blockIdx.x, t = threadIdx.x;
    const int v = blk_node[b];
    const int64_t s0 = blk_start[b], e0 = blk_end[b];
    const int64_t f = first[v], c = count[v], nl = (c + 1) / 2;
    const int ax = node_axis(L, n, xr, f, c);
    if (t == 0 && s0 == f)
        axis_out[v] = ax;
    const uint32_t *La = L + ax * n;
    uint32_t r[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k)
        r[k] = La[min(s0 + t + k * LVL_THREADS, e0 - 1)];
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int64_t p = s0 + t + k * LVL_THREADS;
        if (p < e0)
            byrank[r[k]] = p - f < nl ? 1 : 0;
    }
}

// The sides by rank, a bit each instead of a byte.
__global__ __launch_bounds__(256) void k_side_bits(const uint4 *__restrict__ byrank, int64_t nw,
                                                   uint32_t *bits)
{
    const int64_t i = blockIdx.x * (int64_t)256 + threadIdx.x;
    if (i >= nw)
        return;
    const uint4 a = byrank[2 * i], b = byrank[2 * i + 1];
    const uint32_t w[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
    uint32_t m = 0;
#pragma unroll
    for (int k = 0; k < 8; ++k)  // byte j of a word to bit j
        m |= (((w[k] & 0x01010101u) * 0x01020408u) >> 24 & 0xfu) << (4 * k);
    bits[i] = m;
}

// Sides of a chunk of one list from the sides by rank (stored per position
// for the scatter) and the chunk's left count.
template <bool BITS>
__global__ __launch_bounds__(LVL_THREADS) void k_lvl_count_byrank(
    const uint32_t *__restrict__ L, int64_t n, const int32_t *blk_node,
    const int32_t *blk_start, const int32_t *blk_end, const int32_t *first,
    const int32_t *count, const int32_t *__restrict__ axis, const uint8_t *__restrict__ byrank,
    uint8_t *side, int32_t *cnt, int stride)
{
    constexpr int PER = LVL_CHUNK / LVL_THREADS;
    __shared__ uint32_t sh[8];
    const int b = blockIdx.x, d = blockIdx.y, t = threadIdx.x;
    const int v = blk_node[b];
    const int64_t s0 = blk_start[b], e0 = blk_end[b];
    const int64_t f = first[v], nl = (count[v] + 1) / 2;
    const int ax = axis[v];
    uint32_t g[PER];
    if (d == ax) {
#pragma unroll
        for (int k = 0; k < PER; ++k)
            g[k] = s0 + t + k * LVL_THREADS - f < nl ? 1u : 0u;
    } else {
        const uint32_t *Ld = L + d * n;
        uint32_t r[PER];
#pragma unroll
        for (int k = 0; k < PER; ++k)
            r[k] = Ld[min(s0 + t + k * LVL_THREADS, e0 - 1)];
#pragma unroll
        for (int k = 0; k < PER; ++k)
            g[k] = BITS ? ((const uint32_t *)byrank)[r[k] >> 5] >> (r[k] & 31) & 1u
                        : byrank[r[k]];
    }
    uint8_t *sd = side + d * n;
    uint32_t c = 0;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int64_t p = s0 + t + k * LVL_THREADS;
        if (p < e0) {
            sd[p] = (uint8_t)g[k];
            c += g[k];
        }
    }
    uint32_t total;
    block_excl_scan_u32(c, sh, total);
    if (t == 0)
        cnt[d * stride + b] = (int32_t)total;
}

// Stable partition of one chunk of one list: the chunk is staged in LDS,
// each thread ranks PER consecutive entries, the chunk's left and right runs
// are assembled in LDS and written out as two contiguous runs.
__global__ __launch_bounds__(LVL_THREADS) void k_lvl_scatter(
    const uint32_t *__restrict__ Lsrc, uint32_t *Ldst, int64_t n, const uint8_t *__restrict__ side,
    const int32_t *blk_node, const int32_t *blk_start, const int32_t *blk_end,
    const int32_t *blk_first, const int32_t *first, const int32_t *count, const int32_t *cnt,
    int stride)
{
    constexpr int PER = LVL_CHUNK / LVL_THREADS;
    __shared__ uint32_t sh[8];
    __shared__ uint32_t sv[LVL_CHUNK];
    __shared__ uint32_t so[LVL_CHUNK];
    __shared__ uint8_t sf[LVL_CHUNK];
    const int b = blockIdx.x, d = blockIdx.y, t = threadIdx.x;
    const int v = blk_node[b];
    const int64_t f = first[v], nl = (count[v] + 1) / 2;
    const int64_t s = blk_start[b];
    const int len = (int)(blk_end[b] - s);
    const uint32_t *Ls = Lsrc + d * n + s;
    const uint8_t *sd = side + d * n + s;
    uint32_t *Ld = Ldst + d * n;
    uint32_t part = 0;
    {
        uint32_t lv[PER];
        uint8_t lf[PER];
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const int i = min(t + k * LVL_THREADS, len - 1);  // len >= 1
            lv[k] = Ls[i];
            lf[k] = sd[i];
        }
        // left entries of the node before this chunk: the counts of the
        // node's earlier chunks, loaded while the chunk is in flight
        for (int j = blk_first[b] + t; j < b; j += LVL_THREADS)
            part += (uint32_t)cnt[d * stride + j];
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const int i = t + k * LVL_THREADS;
            if (i < len) {
                sv[i] = lv[k];
                sf[i] = lf[k];
            }
        }
    }
    __syncthreads();
    uint32_t fl[PER];
    uint32_t mine = 0;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int i = t * PER + k;
        fl[k] = i < len ? sf[i] : 0u;
        mine += fl[k];
    }
    uint32_t nleft;
    uint32_t lx = block_excl_scan_u32(mine, sh, nleft);
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int i = t * PER + k;
        if (i < len) {
            const uint32_t pos = fl[k] ? lx : nleft + (uint32_t)i - lx;
            so[pos] = sv[i];
            lx += fl[k];
        }
    }
    __syncthreads();
    // then the two runs
    uint32_t before;
    block_excl_scan_u32(part, sh, before);
    const int64_t nb = (int64_t)before;
    const int64_t lbase = f + nb, rbase = f + nl + (s - f - nb);
    for (int i = t; i < len; i += LVL_THREADS)
        Ld[i < (int)nleft ? lbase + i : rbase + (i - (int)nleft)] = so[i];
}

// ---------------------------------------------------------------- LDS subtrees
// All levels below a cell of at most SUBTREE_MAX particles, by one workgroup.
// A chain of short dependent steps bounds it (a workgroup takes the same time
// alone on the chip as among thousands), so a level is four barriers and no
// search or global load in the chain:
//   - the cell of a position follows from the split rule alone (the left child
//     takes the first ceil(c / 2) positions), so each thread keeps the cells
//     of its positions in registers, and per-cell values are kept at the
//     cell's first position;
//   - coordinates are staged in LDS (the ends of the sorted lists give the
//     extents);
//   - the positions of a wavefront are consecutive, so the partition's counts
//     are ballots: one 64-bit word per wavefront and list, whose prefix sums
//     every wavefront takes for itself;
//   - the lists are partitioned in place (entries wait in registers over the
//     barrier), which leaves LDS for two workgroups per CU.
// 37 us for cells of 2048 particles, 23 for 1000, 239 us at 2^22 particles;
// with tables of the cells, binary searches in them and scans of flags it was
// 63, 43 and 556 us.
__global__ __launch_bounds__(SUBTREE_THREADS) void k_subtree(
    const uint32_t *__restrict__ Lall, int64_t n, const double *__restrict__ xr,
    const int32_t *__restrict__ r2o, const int32_t *__restrict__ sub_root,
    const int32_t *__restrict__ first, const int32_t *__restrict__ count,
    const int32_t *__restrict__ right, const int32_t *__restrict__ level, int leaf_size,
    uint16_t *loc, int32_t *perm, int32_t *axis_out)
{
    constexpr int PER = SUBTREE_MAX / SUBTREE_THREADS;  // positions per thread
    constexpr int WORDS = SUBTREE_MAX / 64;
    static_assert(WORDS <= 64, "one lane per word in the prefix sums");
    static_assert(SUBTREE_MAX <= 1 << 15, "node offsets and counts in 16 bits");
    __shared__ uint32_t rk[SUBTREE_MAX];      // Morton ranks by local id
    __shared__ double xyz[3][SUBTREE_MAX];    // coordinates by local id
    __shared__ uint16_t lst[3][SUBTREE_MAX];  // local ids in the order of each axis
    __shared__ uint8_t flg[SUBTREE_MAX];      // by local id: goes to the left child
    __shared__ uint8_t sax[SUBTREE_MAX];      // split axis, at the cell's first position
    __shared__ uint16_t snode[SUBTREE_MAX];   // node id - root, at the cell's first position
    __shared__ uint64_t msk[3][WORDS];        // left-going entries of 64 positions

    const int t = threadIdx.x, w = t >> 6, lane = lane_id();
    const uint64_t lt = lanemask_lt();
    const int root = sub_root[blockIdx.x];
    const int64_t f0 = first[root];
    const int n0 = count[root];
    const uint32_t *L = Lall + (int64_t)(level[root] & 1) * 3 * n;

    // local id: the place in the first axis list; loc[rank] holds it for the
    // ranks of the other two lists (one entry per particle, in global memory)
    uint32_t rd[PER][3];  // ranks of the axis lists at the thread's positions
    int id[PER][3];
    int cf[PER], cn[PER];  // first position and size of the position's cell (0: no position)
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const int p = t + j * SUBTREE_THREADS;
        cf[j] = 0;
        cn[j] = p < n0 ? n0 : 0;
        if (p < n0) {
#pragma unroll
            for (int d = 0; d < 3; ++d)
                rd[j][d] = L[d * n + f0 + p];
            rk[p] = rd[j][0];
            loc[rd[j][0]] = (uint16_t)p;
#pragma unroll
            for (int d = 0; d < 3; ++d)
                xyz[d][p] = xr[d * n + rd[j][0]];
        }
    }
    if (t == 0)
        snode[0] = 0;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const int p = t + j * SUBTREE_THREADS;
        id[j][0] = p < n0 ? p : 0;
#pragma unroll
        for (int d = 1; d < 3; ++d)
            id[j][d] = p < n0 ? loc[rd[j][d]] : 0;
        if (p < n0) {
#pragma unroll
            for (int d = 0; d < 3; ++d)
                lst[d][p] = (uint16_t)id[j][d];
        }
    }
    __syncthreads();

    // mx: the largest cell of the level
    for (int mx = n0; mx > leaf_size; mx = (mx + 1) >> 1) {
        // split axis of each cell, by the thread of its first position
        int rnode[PER];
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            const int p = t + j * SUBTREE_THREADS;
            rnode[j] = 0;
            if (p == cf[j] && cn[j] > leaf_size) {
                const int node = root + snode[p];
                rnode[j] = right[node] - root;
                int ax = 0;
                double best = 0.0;
#pragma unroll
                for (int d = 0; d < 3; ++d) {
                    const double e = xyz[d][lst[d][p + cn[j] - 1]] - xyz[d][id[j][d]];
                    if (d == 0 || e > best) {
                        best = e;
                        ax = d;
                    }
                }
                sax[p] = (uint8_t)ax;
                axis_out[node] = ax;
            }
        }
        __syncthreads();
        // sides, by local id, from the split axis's list
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            if (cn[j] > leaf_size) {
                const int p = t + j * SUBTREE_THREADS;
                const int ax = sax[cf[j]];
                const int me = ax == 0 ? id[j][0] : (ax == 1 ? id[j][1] : id[j][2]);
                flg[me] = (uint8_t)(p - cf[j] < ((cn[j] + 1) >> 1));
            }
        }
        __syncthreads();
        uint64_t m[PER][3];
#pragma unroll
        for (int j = 0; j < PER; ++j)
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                const bool left = cn[j] > leaf_size && flg[id[j][d]];
                m[j][d] = __ballot(left);
                if (lane == 0)
                    msk[d][w + j * (SUBTREE_THREADS / 64)] = m[j][d];
            }
        __syncthreads();
        // left-going entries before each word, 16 bits per list
        uint64_t pre = 0;
        if (lane < WORDS)
            pre = (uint64_t)__popcll(msk[0][lane]) | ((uint64_t)__popcll(msk[1][lane]) << 16) |
                  ((uint64_t)__popcll(msk[2][lane]) << 32);
        const uint64_t own = pre;
#pragma unroll
        for (int off = 1; off < WORDS; off <<= 1) {
            const uint64_t o = __shfl_up(pre, off);
            if (lane >= off)
                pre += o;
        }
        pre -= own;
        // stable partition; cells that are leaves stay as they are
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            const int p = t + j * SUBTREE_THREADS;
            const int f = cf[j], c = cn[j], nl = (c + 1) >> 1;
            const uint64_t rel = __shfl(pre, w + j * (SUBTREE_THREADS / 64)) - __shfl(pre, f >> 6);
            if (c > leaf_size) {
                const uint64_t below = (1ull << (f & 63)) - 1ull;
#pragma unroll
                for (int d = 0; d < 3; ++d) {
                    const int nb = (int)(int16_t)(rel >> (16 * d)) + __popcll(m[j][d] & lt) -
                                   __popcll(msk[d][f >> 6] & below);
                    const int pos = (m[j][d] >> lane) & 1ull ? f + nb : f + nl + (p - f - nb);
                    lst[d][pos] = (uint16_t)id[j][d];
                }
                if (p == f) {
                    snode[f] += 1;  // cells are numbered in pre-order
                    snode[f + nl] = (uint16_t)rnode[j];
                }
                if (p < f + nl) {
                    cn[j] = nl;
                } else {
                    cf[j] = f + nl;
                    cn[j] = c - nl;
                }
            }
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < PER; ++j)
            if (cn[j] > 0)
#pragma unroll
                for (int d = 0; d < 3; ++d)
                    id[j][d] = lst[d][t + j * SUBTREE_THREADS];
    }

    // leaves: members in ascending Morton rank
    uint32_t me[PER];
    int32_t out[PER];
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        me[j] = rk[id[j][0]];
        out[j] = cn[j] > 0 ? r2o[me[j]] : 0;
    }
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        int rank = 0;
        for (int q = 0; q < cn[j]; ++q)
            rank += rk[lst[0][cf[j] + q]] < me[j];
        if (cn[j] > 0)
            perm[f0 + cf[j] + rank] = out[j];
    }
}

// ---------------------------------------------------------------- driver
// Bounding box (with the non-finite check) and the Morton order: caller
// indices in ascending Morton rank in vals0.
hipError_t launch_morton_order(Tree &t, const double *x, hipStream_t s)
{
    const int64_t n = t.topo.n;
    if (n <= COUNT_SORT_MAX) {
        k_morton_few<<<1, CR_THREADS, 0, s>>>(x, (int)n, t.bbox, t.keys0, t.run_cnt + 2, t.err);
        k_rank_morton<<<(int)((n + 63) / 64), CR_THREADS, 0, s>>>(
            t.keys0, x, (int)n, t.vals0, nullptr, nullptr, nullptr);
        return hipGetLastError();
    }
    const int gs = (int)std::min<int64_t>((n + 255) / 256, 2048);
    k_bbox_init<<<1, 64, 0, s>>>(t.bbox, t.err);
    k_bbox<<<(int)std::min<int64_t>((n + 1023) / 1024, 1024), 256, 0, s>>>(x, n, t.bbox, t.err);
    // Morton keys in (keys1, vals1) -> sorted into (keys0, vals0)
    k_morton<<<gs, 256, 0, s>>>(x, n, t.bbox, t.keys1, t.vals1);
    if (t.morton_full) {
        // concentrated data with distant outliers: most keys share their high
        // half, so the run fix would sort long runs one workgroup each; all
        // eight digits device-wide give the same (key, position) order
        hipError_t e = radix_sort_u64(t.keys1, t.vals1, t.keys0, t.vals0, n, 1, 8, t.rs_hist,
                                      t.rs_tot, s, 8);
        if (e == hipSuccess)
            e = hipMemcpyAsync(t.vals0, t.vals1, n * sizeof(uint32_t), hipMemcpyDeviceToDevice, s);
        return e;
    }
    return sort_by_halves(t.keys1, t.vals1, t.keys0, t.vals1 + n, t.vals0, n, 1, t.rs_hist,
                          t.rs_tot, t.run_cnt + 2, t.run_list, t.err, s);
}

hipError_t launch_build(Tree &t, const double *x, hipStream_t s)
{
    const Topology &T = t.topo;
    const int64_t n = T.n;
    const int gs = (int)std::min<int64_t>((n + 255) / 256, 2048);
    // the two buffers of the axis lists
    uint32_t *L0 = t.lists, *L1 = t.lists + 3 * n;
    if (n <= COUNT_SORT_MAX) {
        const int g = (int)((n + 63) / 64);
        k_morton_few<<<1, CR_THREADS, 0, s>>>(x, (int)n, t.bbox, t.keys0, t.run_cnt + 2, t.err);
        k_rank_morton<<<g, CR_THREADS, 0, s>>>(t.keys0, x, (int)n, t.vals0, t.r2o, t.xr, t.keys1);
        k_rank_axes<<<dim3(g, 3), CR_THREADS, 0, s>>>(t.keys1, (int)n, L0);
    } else {
        hipError_t e = launch_morton_order(t, x, s);
        if (e != hipSuccess)
            return e;
        k_rank_gather<<<gs, 256, 0, s>>>(x, n, t.vals0, t.r2o, t.xr, t.keys1, t.vals1);
        // the three axis arrays (keys1, vals1), the values being the Morton
        // ranks -> the axis lists
        e = sort_by_halves(t.keys1, t.vals1, t.keys0, t.vals0, L0, n, 3, t.rs_hist, t.rs_tot,
                           t.run_cnt, t.run_list, t.err, s);
        if (e != hipSuccess)
            return e;
    }
    for (int l = 0; l < T.nlevels_up; ++l) {
        int b0 = T.lvl_blk_off[l], nb = T.lvl_blk_off[l + 1] - b0;
        const uint32_t *Ls = (l & 1) ? L1 : L0;
        uint32_t *Ld = (l & 1) ? L0 : L1;
        if (n >= LVL_BYRANK_MIN) {
            uint8_t *byrank = (uint8_t *)t.keys0;  // (the sorts are done)
            k_lvl_side<<<nb, LVL_THREADS, 0, s>>>(Ls, n, t.xr, t.blk_node + b0,
                                                  t.blk_start + b0, t.blk_end + b0, t.first,
                                                  t.count, t.axis, byrank);
            const bool bits = n > LVL_BITS_ABOVE;
            const int64_t nw = (n + 31) / 32;
            if (bits)
                k_side_bits<<<(int)((nw + 255) / 256), 256, 0, s>>>((const uint4 *)byrank, nw,
                                                                    (uint32_t *)t.keys1);
            (bits ? k_lvl_count_byrank<true> : k_lvl_count_byrank<false>)
                <<<dim3(nb, 3), LVL_THREADS, 0, s>>>(
                    Ls, n, t.blk_node + b0, t.blk_start + b0, t.blk_end + b0, t.first, t.count,
                    t.axis, bits ? (const uint8_t *)t.keys1 : byrank, t.side, t.lvl_cnt,
                    T.max_lvl_blocks);
        } else {
            k_lvl_count<<<dim3(nb, 3), LVL_THREADS, 0, s>>>(
                Ls, n, t.xr, t.blk_node + b0, t.blk_start + b0, t.blk_end + b0, t.first,
                t.count, t.axis, t.side, t.lvl_cnt, T.max_lvl_blocks);
        }
        k_lvl_scatter<<<dim3(nb, 3), LVL_THREADS, 0, s>>>(
            Ls, Ld, n, t.side, t.blk_node + b0, t.blk_start + b0, t.blk_end + b0,
            t.blk_first + b0, t.first, t.count, t.lvl_cnt, T.max_lvl_blocks);
    }
    int nsub = (int)T.sub_root.size();
    k_subtree<<<nsub, SUBTREE_THREADS, 0, s>>>(t.lists, n, t.xr, t.r2o, t.sub_root, t.first,
                                               t.count, t.right, t.level, T.leaf_size,
                                               (uint16_t *)t.side, t.perm, t.axis);
    return hipGetLastError();
}

}  // namespace fmm
