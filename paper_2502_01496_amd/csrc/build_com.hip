// kd-tree cut through the centre of mass (FMM_TREE_COM) on gfx950.
//
// Sec. 2 describes the tree as cut recursively through each cell's centre of
// mass across its longest axis, down to cells of at most leaf_size
// particles.  Positions are quantised on a grid of 2^32 steps over the
// largest extent of the global bounding box and masses to integer weights
// (w = floor(m / m_max 2^24) in [1, 2^24]); per cell the axis is the longest
// of the quantised bounding box (ties -> lowest) and a particle goes left iff
// q_d sum(w) < sum(w q_d).  All of it is integer arithmetic, so the partition
// does not depend on how the sums are split over threads.  A cell whose
// particles share one grid point is halved in tree order.
//
// The shape depends on the data, so the build is level-synchronous over the
// cells of more than COM_SUB particles ("active"), each cut in chunks of
// COM_CHUNK particles:
//   stats (per chunk: quantised box, sum w, sum w q) -> count (per chunk: its
//   cell's stats folded, axis and cut, particles going left) -> scatter (per
//   chunk: stable partition into the other buffer; the two new cells) -> next
//   (one workgroup: the next level's active cells and chunks).
// The sizes of a level stay on the device; the host launches the levels that a
// balanced tree has and reads back once, then one by one while cells are left.
// Every cell of at most COM_SUB particles is finished by one workgroup in LDS
// (all levels below it).  Cells are numbered as they appear and renumbered to
// DFS pre-order: a finished cell's nodes among themselves in LDS, the cells
// above by one workgroup.  The internal cells by level follow from one pass of
// the radix sort.
// Launches bound the build at a few 10^5 particles: 200003 (leaf 10) took 1.57
// ms as 18 levels of 8 launches and a readback each, this 0.54; 2^20 particles
// 3.68 and 1.12 ms.
#include "fmm_internal.h"

namespace fmm {

constexpr int CB = 1024;  // threads per chunk workgroup
constexpr int COM_SUB = 2048;  // largest cell finished in LDS

// control words: active cells and chunks of the level, finished cells, m_max
// bits, cells so far, levels above the finished cells, cells and leaves in
// all, depth, large cells (written, counted), then internal cells per level
enum { CA = 0, CC = 1, CS = 2, CMM = 3, CNN = 4, CLEV = 5, CTOT = 6, CLEAF = 7, CDEP = 8, CBIG = 9,
       CNBIG = 10, CLVL = 16 };
static_assert(CLVL + COM_MAX_DEPTH <= COM_CTL, "control words");

// node table rows of the cells above the finished ones, and of those: first,
// count, parent, level, axis, children, pre-order id
enum { NF = 0, NC = 1, NP = 2, NLV = 3, NAX = 4, NL = 5, NR = 6, NPRE = 7 };
// renumbering rows: nodes of the subtree, leaves before it, first cell of each
// level, finished cells
enum { RSUB = 0, RLOFS = 1, RLEV = 2, RFIN = 3 };

__device__ __forceinline__ void add128(uint64_t &lo, uint64_t &hi, uint64_t blo, uint64_t bhi)
{
    const uint64_t s = lo + blo;
    hi += bhi + (s < lo ? 1ull : 0ull);
    lo = s;
}

// q_d sum(w) < sum(w q_d), both sides exact 128-bit integers
__device__ __forceinline__ bool left_of_cut(uint32_t qd, uint64_t sw, uint64_t lo, uint64_t hi)
{
    const uint64_t plo = (uint64_t)qd * sw;
    const uint64_t phi = __umul64hi((uint64_t)qd, sw);
    return phi < hi || (phi == hi && plo < lo);
}

__global__ void k_com_zero(int64_t *ctl)
{
    if (threadIdx.x < COM_CTL)
        ctl[threadIdx.x] = 0;
}

// Largest positive mass (NaN and non-positive masses ignored), as ordered
// bits in ctl[CMM]; one atomic per workgroup.
__global__ __launch_bounds__(256) void k_com_mmax(const double *__restrict__ m, int64_t n,
                                                  int64_t *ctl)
{
    __shared__ uint64_t sh[4];
    uint64_t best = 0ull;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        const double v = m[i];
        if (v > 0.0) {
            const uint64_t b = ordbits(v);
            best = b > best ? b : best;
        }
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        const uint64_t o = __shfl_xor((unsigned long long)best, off);
        best = o > best ? o : best;
    }
    if (lane_id() == 0)
        sh[threadIdx.x >> 6] = best;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < 4; ++w)
            best = sh[w] > best ? sh[w] : best;
        if (best)
            atomicMax((unsigned long long *)&ctl[CMM], (unsigned long long)best);
    }
}

// Tree order = Morton order; quantised coordinates and weights.
__global__ __launch_bounds__(256) void k_com_init(const double *__restrict__ x,
                                                  const double *__restrict__ m, int64_t n,
                                                  const uint64_t *__restrict__ bbox,
                                                  const int64_t *__restrict__ ctl,
                                                  const uint32_t *__restrict__ order,
                                                  int32_t *perm, uint32_t *q)
{
    double lo[3], ext = 0.0;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        lo[d] = from_ordbits(bbox[d]);
        const double e = from_ordbits(bbox[3 + d]) - lo[d];
        if (e > ext)
            ext = e;
    }
    if (ext == 0.0)
        ext = 1.0;
    const double scale = 4294967296.0 / ext;
    const uint64_t mb = (uint64_t)ctl[CMM];
    const double mmax = mb ? from_ordbits(mb) : 0.0;
    for (int64_t p = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; p < n;
         p += (int64_t)gridDim.x * blockDim.x) {
        const int64_t i = order[p];
        perm[p] = (int32_t)i;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            const double v = floor((x[3 * i + d] - lo[d]) * scale);
            q[d * n + p] = v >= 4294967295.0 ? 4294967295u : (v >= 0.0 ? (uint32_t)v : 0u);
        }
        uint32_t w = 1u;
        if (m && mmax > 0.0) {
            const double v = floor(m[i] / mmax * 16777216.0);
            w = v >= 1.0 ? (v <= 16777216.0 ? (uint32_t)v : 16777216u) : 1u;
        }
        q[3 * n + p] = w;
    }
}

// The root cell and, when it is active, its chunks.
__global__ __launch_bounds__(256) void k_com_root(int64_t n, int32_t *node, int64_t cap,
                                                  int32_t *act, int64_t *choff, int32_t *chk,
                                                  int64_t cap_c, int32_t *ren, int64_t *ctl)
{
    const int t = threadIdx.x;
    const bool cut = n > COM_SUB;
    const int64_t nch = cut ? (n + COM_CHUNK - 1) / COM_CHUNK : 0;
    if (t == 0) {
        node[NF * cap] = 0;
        node[NC * cap] = (int32_t)n;
        node[NP * cap] = -1;
        node[NLV * cap] = 0;
        node[NAX * cap] = -1;
        node[NL * cap] = -1;
        node[NR * cap] = -1;
        act[0] = 0;
        choff[0] = 0;
        choff[1] = nch;
        ren[RLEV * cap] = 0;
        ren[RFIN * cap] = 0;
        ctl[CA] = cut ? 1 : 0;
        ctl[CC] = nch;
        ctl[CS] = cut ? 0 : 1;
        ctl[CNN] = 1;
        ctl[CLEV] = 1;
    }
    for (int64_t c = t; c < nch; c += blockDim.x) {
        chk[c] = 0;
        chk[cap_c + c] = (int32_t)(c * COM_CHUNK);
        chk[2 * cap_c + c] = (int32_t)std::min<int64_t>(n, (c + 1) * COM_CHUNK);
    }
}

// Per chunk: quantised box, sum w and sum w q_d (d = 0..2, 128-bit).
__global__ __launch_bounds__(CB) void k_com_stats(const uint32_t *__restrict__ q, int64_t n,
                                                  const int32_t *__restrict__ chk, int64_t cap_c,
                                                  uint64_t *cpart,
                                                  const int64_t *__restrict__ ctl)
{
    __shared__ uint64_t sh[CB / 64][13];
    const int c = blockIdx.x;
    if (c >= ctl[CC])
        return;
    const int start = chk[cap_c + c], end = chk[2 * cap_c + c];
    uint32_t mn[3] = {~0u, ~0u, ~0u}, mx[3] = {0u, 0u, 0u};
    uint64_t sw = 0ull, lo[3] = {0ull, 0ull, 0ull}, hi[3] = {0ull, 0ull, 0ull};
    for (int p = start + threadIdx.x; p < end; p += CB) {
        const uint64_t w = q[3 * n + p];
        sw += w;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            const uint32_t v = q[d * n + p];
            mn[d] = v < mn[d] ? v : mn[d];
            mx[d] = v > mx[d] ? v : mx[d];
            add128(lo[d], hi[d], w * (uint64_t)v, 0ull);
        }
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        sw += __shfl_xor((unsigned long long)sw, off);
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            const uint32_t a = (uint32_t)__shfl_xor((int)mn[d], off);
            const uint32_t b = (uint32_t)__shfl_xor((int)mx[d], off);
            mn[d] = a < mn[d] ? a : mn[d];
            mx[d] = b > mx[d] ? b : mx[d];
            const uint64_t ol = __shfl_xor((unsigned long long)lo[d], off);
            const uint64_t oh = __shfl_xor((unsigned long long)hi[d], off);
            add128(lo[d], hi[d], ol, oh);
        }
    }
    const int wv = threadIdx.x >> 6;
    if (lane_id() == 0) {
        for (int d = 0; d < 3; ++d) {
            sh[wv][d] = mn[d];
            sh[wv][3 + d] = mx[d];
            sh[wv][7 + 2 * d] = lo[d];
            sh[wv][8 + 2 * d] = hi[d];
        }
        sh[wv][6] = sw;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        uint64_t r[13];
        for (int k = 0; k < 13; ++k)
            r[k] = sh[0][k];
        for (int w = 1; w < CB / 64; ++w) {
            for (int d = 0; d < 3; ++d) {
                r[d] = sh[w][d] < r[d] ? sh[w][d] : r[d];
                r[3 + d] = sh[w][3 + d] > r[3 + d] ? sh[w][3 + d] : r[3 + d];
                add128(r[7 + 2 * d], r[8 + 2 * d], sh[w][7 + 2 * d], sh[w][8 + 2 * d]);
            }
            r[6] += sh[w][6];
        }
        uint64_t *o = cpart + 16 * (int64_t)c;
        for (int k = 0; k < 13; ++k)
            o[k] = r[k];
    }
}

__device__ __forceinline__ bool goes_left(const uint32_t *__restrict__ q, int64_t n, int p,
                                          int first, int count, const uint64_t *sp)
{
    const int ax = (int)(sp[0] & 0xffull);
    if (sp[0] >> 8)
        return p - first < (count + 1) / 2;  // one grid point: halve in tree order
    return left_of_cut(q[ax * n + p], sp[1], sp[2], sp[3]);
}

// Per chunk: the cell's chunks folded; axis, degenerate flag and cut (split[4a]
// = axis | degenerate << 8, then sum w, sum w q_axis (lo, hi), written by the
// cell's first chunk); particles going left.
__global__ __launch_bounds__(CB) void k_com_count(const uint32_t *__restrict__ q, int64_t n,
                                                  const int32_t *__restrict__ chk, int64_t cap_c,
                                                  const int32_t *__restrict__ act,
                                                  const int64_t *__restrict__ choff,
                                                  const int32_t *__restrict__ node, int64_t cap,
                                                  const uint64_t *__restrict__ cpart,
                                                  uint64_t *split, int32_t *cleft,
                                                  const int64_t *__restrict__ ctl)
{
    __shared__ uint64_t sp[4];
    __shared__ int sh[CB / 64];
    const int c = blockIdx.x;
    if (c >= ctl[CC])
        return;
    const int a = chk[c], start = chk[cap_c + c], end = chk[2 * cap_c + c];
    const int v = act[a];
    const int f = node[NF * cap + v], cnt = node[NC * cap + v];
    if (threadIdx.x < 64) {
        uint64_t mn[3] = {~0ull, ~0ull, ~0ull}, mx[3] = {0ull, 0ull, 0ull};
        uint64_t sw = 0ull, lo[3] = {0ull, 0ull, 0ull}, hi[3] = {0ull, 0ull, 0ull};
        for (int64_t j = choff[a] + threadIdx.x; j < choff[a + 1]; j += 64) {
            const uint64_t *r = cpart + 16 * j;
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                mn[d] = r[d] < mn[d] ? r[d] : mn[d];
                mx[d] = r[3 + d] > mx[d] ? r[3 + d] : mx[d];
                add128(lo[d], hi[d], r[7 + 2 * d], r[8 + 2 * d]);
            }
            sw += r[6];
        }
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) {
            sw += __shfl_xor((unsigned long long)sw, off);
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                const uint64_t x = __shfl_xor((unsigned long long)mn[d], off);
                const uint64_t y = __shfl_xor((unsigned long long)mx[d], off);
                mn[d] = x < mn[d] ? x : mn[d];
                mx[d] = y > mx[d] ? y : mx[d];
                const uint64_t ol = __shfl_xor((unsigned long long)lo[d], off);
                const uint64_t oh = __shfl_xor((unsigned long long)hi[d], off);
                add128(lo[d], hi[d], ol, oh);
            }
        }
        if (threadIdx.x == 0) {
            int ax = 0;
            uint64_t ext = mx[0] - mn[0], slo = lo[0], shi = hi[0];
#pragma unroll
            for (int d = 1; d < 3; ++d)
                if (mx[d] - mn[d] > ext) {
                    ax = d;
                    ext = mx[d] - mn[d];
                    slo = lo[d];
                    shi = hi[d];
                }
            sp[0] = (uint64_t)ax | (ext == 0ull ? 1ull << 8 : 0ull);
            sp[1] = sw;
            sp[2] = slo;
            sp[3] = shi;
            if (c == choff[a])
                for (int k = 0; k < 4; ++k)
                    split[4 * (int64_t)a + k] = sp[k];
        }
    }
    __syncthreads();
    int k = 0;
    for (int p = start + threadIdx.x; p < end; p += CB)
        k += goes_left(q, n, p, f, cnt, sp) ? 1 : 0;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1)
        k += __shfl_xor(k, off);
    if (lane_id() == 0)
        sh[threadIdx.x >> 6] = k;
    __syncthreads();
    if (threadIdx.x == 0) {
        int tot = 0;
        for (int w = 0; w < CB / 64; ++w)
            tot += sh[w];
        cleft[c] = tot;
    }
}

// Per chunk: stable partition into the other buffer, CB particles per round in
// order (a round's lanes hold consecutive particles).  The cell's first chunk
// writes its children: cells NN + 2a (left) and NN + 2a + 1 (right).
__global__ __launch_bounds__(CB) void k_com_scatter(
    const uint32_t *__restrict__ q, const int32_t *__restrict__ perm, int64_t n,
    const int32_t *__restrict__ chk, int64_t cap_c, const int32_t *__restrict__ act,
    const int64_t *__restrict__ choff, int32_t *node, int64_t cap,
    const uint64_t *__restrict__ split, const int32_t *__restrict__ cleft, uint32_t *q_out,
    int32_t *perm_out, const int64_t *__restrict__ ctl)
{
    __shared__ int wl[CB / 64];
    __shared__ int sbase[2];
    const int c = blockIdx.x;
    if (c >= ctl[CC])
        return;
    const int a = chk[c], start = chk[cap_c + c], end = chk[2 * cap_c + c];
    const int v = act[a];
    const int f = node[NF * cap + v], cnt = node[NC * cap + v];
    const uint64_t *sp = split + 4 * (int64_t)a;
    if (threadIdx.x < 64) {
        // left particles of the cell's earlier chunks, and of all
        int before = 0, all = 0;
        for (int64_t j = choff[a] + threadIdx.x; j < choff[a + 1]; j += 64) {
            const int l = cleft[j];
            all += l;
            before += j < c ? l : 0;
        }
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) {
            before += __shfl_xor(before, off);
            all += __shfl_xor(all, off);
        }
        if (threadIdx.x == 0) {
            sbase[0] = before;
            sbase[1] = all;
            if (c == choff[a]) {
                const int l = (int)ctl[CNN] + 2 * a, r = l + 1, lv = node[NLV * cap + v] + 1;
                node[NF * cap + l] = f;
                node[NF * cap + r] = f + all;
                node[NC * cap + l] = all;
                node[NC * cap + r] = cnt - all;
                for (int u = l; u <= r; ++u) {
                    node[NP * cap + u] = v;
                    node[NLV * cap + u] = lv;
                    node[NAX * cap + u] = -1;
                    node[NL * cap + u] = -1;
                    node[NR * cap + u] = -1;
                }
                node[NL * cap + v] = l;
                node[NR * cap + v] = r;
                node[NAX * cap + v] = (int)(sp[0] & 0xffull);
            }
        }
    }
    __syncthreads();
    int bl = f + sbase[0], br = f + sbase[1] + (start - f - sbase[0]);
    const int wv = threadIdx.x >> 6;
    const uint64_t lt = lanemask_lt();
    for (int r0 = start; r0 < end; r0 += CB) {
        const int p = r0 + threadIdx.x;
        const bool valid = p < end;
        const bool left = valid && goes_left(q, n, p, f, cnt, sp);
        const uint64_t bal = __ballot(left);
        if (lane_id() == 0)
            wl[wv] = __popcll(bal);
        __syncthreads();
        int before = 0, total = 0;
        for (int w = 0; w < CB / 64; ++w) {
            before += w < wv ? wl[w] : 0;
            total += wl[w];
        }
        const int rank_l = before + __popcll(bal & lt);
        if (valid) {
            const int dst = left ? bl + rank_l : br + ((int)threadIdx.x - rank_l);
#pragma unroll
            for (int d = 0; d < 4; ++d)
                q_out[d * n + dst] = q[d * n + p];
            perm_out[dst] = perm[p];
        }
        const int nvalid = min(CB, end - r0);
        bl += total;
        br += nvalid - total;
        __syncthreads();
    }
}

// One workgroup: over the children of the level's active cells, the next
// level's active cells with their chunks, and the others appended to the cells
// to be finished.
constexpr int NEXT_T = 1024;

__device__ __forceinline__ int block_excl_scan(int v, int *sh, int &total)
{
    // inclusive scan within waves, then over the wave sums
    const int lane = lane_id(), wv = threadIdx.x >> 6;
    int x = v;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int y = __shfl_up(x, off);
        if (lane >= off)
            x += y;
    }
    if (lane == 63)
        sh[wv] = x;
    __syncthreads();
    if (threadIdx.x == 0) {
        int run = 0;
        for (int w = 0; w < NEXT_T / 64; ++w) {
            const int t = sh[w];
            sh[w] = run;
            run += t;
        }
        sh[NEXT_T / 64] = run;
    }
    __syncthreads();
    const int ex = sh[wv] + x - v;
    total = sh[NEXT_T / 64];
    __syncthreads();
    return ex;
}

__global__ __launch_bounds__(NEXT_T) void k_com_next(int level, const int32_t *__restrict__ node,
                                                    int64_t cap, int32_t *act, int64_t *choff,
                                                    int32_t *chk, int64_t cap_c, int32_t *ren,
                                                    int64_t *ctl)
{
    __shared__ int sh[NEXT_T / 64 + 1];
    const int NN = (int)ctl[CNN], m = 2 * (int)ctl[CA];
    int base_a = 0, base_s = (int)ctl[CS];
    int64_t base_c = 0;
    for (int k0 = 0; k0 < m; k0 += NEXT_T) {
        const int k = k0 + threadIdx.x;
        const int u = NN + k;
        const int cnt = k < m ? node[NC * cap + u] : 0;
        const int isact = cnt > COM_SUB ? 1 : 0;
        const int nch = isact ? (cnt + COM_CHUNK - 1) / COM_CHUNK : 0;
        const int isfin = k < m && !isact ? 1 : 0;
        int ta, tc, ts;
        const int pa = block_excl_scan(isact, sh, ta);
        const int pc = block_excl_scan(nch, sh, tc);
        const int ps = block_excl_scan(isfin, sh, ts);
        if (isact) {
            const int ai = base_a + pa;
            const int64_t c0 = base_c + pc;
            act[ai] = u;
            choff[ai] = c0;
            const int f = node[NF * cap + u];
            for (int j = 0; j < nch; ++j) {
                chk[c0 + j] = ai;
                chk[cap_c + c0 + j] = f + j * COM_CHUNK;
                chk[2 * cap_c + c0 + j] = f + min(cnt, (j + 1) * COM_CHUNK);
            }
        }
        if (isfin)
            ren[RFIN * cap + base_s + ps] = u;
        base_a += ta;
        base_c += tc;
        base_s += ts;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        choff[base_a] = base_c;
        if (m > 0) {
            ren[RLEV * cap + level + 1] = NN;
            ctl[CLEV] = level + 2;
        }
        ctl[CA] = base_a;
        ctl[CC] = base_c;
        ctl[CS] = base_s;
        ctl[CNN] = NN + m;
    }
}

// A node of a finished cell, in pre-order within it: first position and count,
// distance to the right child (0: a leaf) and to the parent, axis, level, all
// relative to the cell.
__device__ __forceinline__ uint64_t fin_pack(int f, int c, int right, int parent, int ax, int lv)
{
    return (uint64_t)f | ((uint64_t)c << 12) | ((uint64_t)right << 24) | ((uint64_t)parent << 36) |
           ((uint64_t)ax << 48) | ((uint64_t)lv << 50);
}

// All levels below a cell of at most COM_SUB particles, one workgroup per cell.
// A wavefront cuts one cell at a time: extents, then the sums of the chosen
// axis, then the partition, 64 particles per round; particles move as local
// ids, between two buffers by level.  Nodes are numbered as they appear (in an
// order that may differ from run to run) and then in pre-order.
constexpr int FIN_T = 1024, FIN_W = FIN_T / 64, FIN_NODES = 2 * COM_SUB;

__global__ __launch_bounds__(FIN_T) void k_com_finish(
    const uint32_t *__restrict__ q0, const int32_t *__restrict__ perm0,
    const uint32_t *__restrict__ q1, const int32_t *__restrict__ perm1, int64_t n,
    const int32_t *__restrict__ node, int64_t cap, int leaf_size, int32_t *ren, uint64_t *rec,
    int32_t *perm_out, int64_t *ctl)
{
    __shared__ uint32_t q[4][COM_SUB];     // coordinates and weight by local id
    __shared__ int32_t pm[COM_SUB];        // caller index by local id
    __shared__ uint16_t idx[2][COM_SUB];   // local ids in tree order
    __shared__ uint16_t nf[FIN_NODES], nc[FIN_NODES], nl[FIN_NODES], np[FIN_NODES];
    __shared__ uint16_t nsub[FIN_NODES], npre[FIN_NODES];
    __shared__ uint8_t nax[FIN_NODES];
    __shared__ uint16_t lev[COM_SUB + 2];  // first node of each level
    __shared__ int nn, nbig;
    __shared__ int lcnt[COM_MAX_DEPTH];    // internal nodes per (absolute) level
    const int t = threadIdx.x, w = t >> 6, lane = lane_id();
    const uint64_t lt = lanemask_lt();
    const int v0 = ren[RFIN * cap + blockIdx.x];
    const int f0 = node[NF * cap + v0], c0 = node[NC * cap + v0], lv0 = node[NLV * cap + v0];
    const uint32_t *qg = lv0 & 1 ? q1 : q0;
    const int32_t *pg = lv0 & 1 ? perm1 : perm0;
    for (int p = t; p < c0; p += FIN_T) {
#pragma unroll
        for (int d = 0; d < 4; ++d)
            q[d][p] = qg[d * n + f0 + p];
        pm[p] = pg[f0 + p];
        idx[0][p] = (uint16_t)p;
    }
    for (int i = t; i < COM_MAX_DEPTH; i += FIN_T)
        lcnt[i] = 0;
    if (t == 0) {
        nf[0] = 0;
        nc[0] = (uint16_t)c0;
        np[0] = 0;
        nn = 1;
        nbig = 0;
        lev[0] = 0;
    }
    __syncthreads();
    int lo = 0, hi = 1, depth = 0;
    while (lo < hi) {
        const int par = depth & 1;
        for (int v = lo + w; v < hi; v += FIN_W) {
            const int f = nf[v], c = nc[v];
            if (c <= leaf_size) {
                for (int i = lane; i < c; i += 64)
                    perm_out[f0 + f + i] = pm[idx[par][f + i]];
                if (lane == 0) {
                    nl[v] = 0;
                    nax[v] = 0;
                    if (c >= 64)
                        atomicAdd(&nbig, 1);
                }
                continue;
            }
            uint32_t mn[3] = {~0u, ~0u, ~0u}, mx[3] = {0u, 0u, 0u};
            for (int i = lane; i < c; i += 64) {
                const int id = idx[par][f + i];
#pragma unroll
                for (int d = 0; d < 3; ++d) {
                    const uint32_t x = q[d][id];
                    mn[d] = x < mn[d] ? x : mn[d];
                    mx[d] = x > mx[d] ? x : mx[d];
                }
            }
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1)
#pragma unroll
                for (int d = 0; d < 3; ++d) {
                    const uint32_t x = (uint32_t)__shfl_xor((int)mn[d], off);
                    const uint32_t y = (uint32_t)__shfl_xor((int)mx[d], off);
                    mn[d] = x < mn[d] ? x : mn[d];
                    mx[d] = y > mx[d] ? y : mx[d];
                }
            int ax = 0;
            uint32_t ext = mx[0] - mn[0];
#pragma unroll
            for (int d = 1; d < 3; ++d)
                if (mx[d] - mn[d] > ext) {
                    ax = d;
                    ext = mx[d] - mn[d];
                }
            // sum w and sum w q of the axis: w q < 2^56, 2^11 terms, summed in
            // two halves
            uint64_t sw = 0, sl = 0, sh = 0;
            for (int i = lane; i < c; i += 64) {
                const int id = idx[par][f + i];
                const uint64_t wt = q[3][id], p = wt * (uint64_t)q[ax][id];
                sw += wt;
                sl += p & 0xffffffffull;
                sh += p >> 32;
            }
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) {
                sw += __shfl_xor((unsigned long long)sw, off);
                sl += __shfl_xor((unsigned long long)sl, off);
                sh += __shfl_xor((unsigned long long)sh, off);
            }
            uint64_t wql = sh << 32, wqh = sh >> 32;
            add128(wql, wqh, sl, 0ull);
            auto left_of = [&](int i, int id) {
                return ext == 0u ? i < (c + 1) / 2 : left_of_cut(q[ax][id], sw, wql, wqh);
            };
            int left = 0;
            for (int i0 = 0; i0 < c; i0 += 64) {
                const int i = i0 + lane;
                left += __popcll(__ballot(i < c && left_of(i, idx[par][f + min(i, c - 1)])));
            }
            int bl = 0;
            for (int i0 = 0; i0 < c; i0 += 64) {
                const int i = i0 + lane;
                const int id = idx[par][f + min(i, c - 1)];
                const uint64_t bal = __ballot(i < c && left_of(i, id));
                const int rank = bl + __popcll(bal & lt);
                if (i < c)
                    idx[par ^ 1][f + ((bal >> lane) & 1ull ? rank : left + i - rank)] =
                        (uint16_t)id;
                bl += __popcll(bal);
            }
            if (lane == 0) {
                const int u = atomicAdd(&nn, 2);
                nl[v] = (uint16_t)u;
                nax[v] = (uint8_t)ax;
                nf[u] = (uint16_t)f;
                nc[u] = (uint16_t)left;
                nf[u + 1] = (uint16_t)(f + left);
                nc[u + 1] = (uint16_t)(c - left);
                np[u] = np[u + 1] = (uint16_t)v;
                if (c >= 64)
                    atomicAdd(&nbig, 1);
                if (lv0 + depth < COM_MAX_DEPTH)
                    atomicAdd(&lcnt[lv0 + depth], 1);
            }
        }
        __syncthreads();
        lo = hi;
        hi = nn;
        ++depth;
        if (t == 0)
            lev[depth] = (uint16_t)lo;
        __syncthreads();
    }
    // subtree sizes from the deepest level up, pre-order ids from the root down
    for (int l = depth - 1; l >= 0; --l) {
        for (int v = lev[l] + t; v < lev[l + 1]; v += FIN_T)
            nsub[v] = nl[v] ? (uint16_t)(1 + nsub[nl[v]] + nsub[nl[v] + 1]) : (uint16_t)1;
        __syncthreads();
    }
    if (t == 0)
        npre[0] = 0;
    __syncthreads();
    for (int l = 0; l < depth; ++l) {
        for (int v = lev[l] + t; v < lev[l + 1]; v += FIN_T) {
            const int u = nl[v], P = npre[v];
            if (u) {
                npre[u] = (uint16_t)(P + 1);
                npre[u + 1] = (uint16_t)(P + 1 + nsub[u]);
            }
            rec[2 * (int64_t)f0 + P] =
                fin_pack(nf[v], nc[v], u ? 1 + nsub[u] : 0, P - npre[np[v]], nax[v], l);
        }
        __syncthreads();
    }
    if (t == 0) {
        ren[RSUB * cap + v0] = nsub[0];
        atomicMax((unsigned long long *)&ctl[CDEP], (unsigned long long)(lv0 + depth));
        atomicAdd((unsigned long long *)&ctl[CNBIG], (unsigned long long)nbig);
    }
    for (int i = t; i < COM_MAX_DEPTH; i += FIN_T)
        if (lcnt[i])
            atomicAdd((unsigned long long *)&ctl[CLVL + i], (unsigned long long)lcnt[i]);
}

// One workgroup: subtree sizes of the cells above the finished ones from the
// deepest level up, then pre-order ids and leaf offsets from the root down (a
// subtree of k nodes has (k + 1) / 2 leaves).
__global__ __launch_bounds__(1024) void k_com_number(int32_t *node, int64_t cap, int32_t *ren,
                                                     int64_t *ctl)
{
    const int nlev = (int)ctl[CLEV], NN = (int)ctl[CNN], t = threadIdx.x;
    auto first_of = [&](int l) { return l < nlev ? ren[RLEV * cap + l] : NN; };
    for (int l = nlev - 1; l >= 0; --l) {
        for (int v = first_of(l) + t; v < first_of(l + 1); v += 1024) {
            const int a = node[NL * cap + v], b = node[NR * cap + v];
            if (a >= 0) {
                ren[RSUB * cap + v] = 1 + ren[RSUB * cap + a] + ren[RSUB * cap + b];
                atomicAdd((unsigned long long *)&ctl[CNBIG], 1ull);
                if (l < COM_MAX_DEPTH)
                    atomicAdd((unsigned long long *)&ctl[CLVL + l], 1ull);
            }
        }
        __syncthreads();
    }
    if (t == 0) {
        node[NPRE * cap] = 0;
        ren[RLOFS * cap] = 0;
        ctl[CTOT] = ren[RSUB * cap];
        ctl[CLEAF] = (ren[RSUB * cap] + 1) / 2;
    }
    __syncthreads();
    for (int l = 0; l < nlev; ++l) {
        for (int v = first_of(l) + t; v < first_of(l + 1); v += 1024) {
            const int a = node[NL * cap + v], b = node[NR * cap + v];
            if (a >= 0) {
                const int P = node[NPRE * cap + v], o = ren[RLOFS * cap + v];
                const int sa = ren[RSUB * cap + a];
                node[NPRE * cap + a] = P + 1;
                node[NPRE * cap + b] = P + 1 + sa;
                ren[RLOFS * cap + a] = o;
                ren[RLOFS * cap + b] = o + (sa + 1) / 2;
            }
        }
        __syncthreads();
    }
}

// The topology arrays at the pre-order ids, the list of large cells, and the
// sort keys of the internal cells by level (leaves last).  Workgroups 0 ..
// nfin - 1: the nodes of a finished cell, the others: the cells above.
struct ComOut {
    int32_t *first, *count, *left, *right, *parent, *level, *axis, *node_leaf, *leaf_node, *big;
    uint32_t *key, *val;
};

__device__ __forceinline__ void com_emit(const ComOut &O, int P, int f, int c, int left, int right,
                                         int parent, int lv, int ax, int leaf, int64_t *ctl)
{
    O.first[P] = f;
    O.count[P] = c;
    O.left[P] = left;
    O.right[P] = right;
    O.parent[P] = parent;
    O.level[P] = lv;
    O.axis[P] = ax;
    O.node_leaf[P] = leaf;
    if (leaf >= 0)
        O.leaf_node[leaf] = P;
    O.key[P] = leaf >= 0 ? 255u : (uint32_t)min(lv, 254);
    O.val[P] = (uint32_t)P;
    if (c >= 64)
        O.big[atomicAdd((unsigned long long *)&ctl[CBIG], 1ull)] = P;
}

__global__ __launch_bounds__(256) void k_com_emit(int nfin, const int32_t *__restrict__ node,
                                                 int64_t cap, const int32_t *__restrict__ ren,
                                                 const uint64_t *__restrict__ rec, ComOut O,
                                                 int64_t *ctl)
{
    const int t = threadIdx.x;
    if ((int)blockIdx.x >= nfin) {
        const int NN = (int)ctl[CNN];
        for (int v = ((int)blockIdx.x - nfin) * 256 + t; v < NN;
             v += ((int)gridDim.x - nfin) * 256) {
            const int a = node[NL * cap + v], b = node[NR * cap + v], pa = node[NP * cap + v];
            if (a >= 0)
                com_emit(O, node[NPRE * cap + v], node[NF * cap + v], node[NC * cap + v],
                         node[NPRE * cap + a], node[NPRE * cap + b],
                         pa >= 0 ? node[NPRE * cap + pa] : -1, node[NLV * cap + v],
                         node[NAX * cap + v], -1, ctl);
        }
        return;
    }
    __shared__ int wl[4];
    const int v = ren[RFIN * cap + blockIdx.x];
    const int P0 = node[NPRE * cap + v], f0 = node[NF * cap + v], lv0 = node[NLV * cap + v];
    const int pa = node[NP * cap + v], k = ren[RSUB * cap + v];
    int lofs = ren[RLOFS * cap + v];
    const uint64_t *r = rec + 2 * (int64_t)f0;
    for (int i0 = 0; i0 < k; i0 += 256) {
        const int i = i0 + t;
        const uint64_t x = i < k ? r[i] : 0ull;
        const int right = (int)(x >> 24) & 0xfff, up = (int)(x >> 36) & 0xfff;
        const bool leaf = i < k && right == 0;
        const uint64_t bal = __ballot(leaf);
        if (lane_id() == 0)
            wl[t >> 6] = __popcll(bal);
        __syncthreads();
        int before = 0, total = 0;
        for (int w = 0; w < 4; ++w) {
            before += w < (t >> 6) ? wl[w] : 0;
            total += wl[w];
        }
        if (i < k) {
            const int P = P0 + i;
            com_emit(O, P, f0 + (int)(x & 0xfff), (int)(x >> 12) & 0xfff, leaf ? -1 : P + 1,
                     leaf ? -1 : P + right, i ? P - up : (pa >= 0 ? node[NPRE * cap + pa] : -1),
                     lv0 + (int)(x >> 50), leaf ? -1 : (int)(x >> 48) & 3,
                     leaf ? lofs + before + __popcll(bal & lanemask_lt()) : -1, ctl);
        }
        lofs += total;
        __syncthreads();
    }
}

static hipError_t read_ctl(Tree &t, hipStream_t s)
{
    hipError_t e = hipMemcpyAsync(t.cw.h_ctl, t.cw.ctl, COM_CTL * sizeof(int64_t),
                                  hipMemcpyDeviceToHost, s);
    if (e == hipSuccess)
        e = hipStreamSynchronize(s);
    return e;
}

int64_t com_max_active(int64_t n) { return n / (COM_SUB + 1) + 1; }

hipError_t launch_build_com(Tree &t, const double *x, const double *m, hipStream_t s)
{
    Topology &T = t.topo;
    Tree::ComWork &W = t.cw;
    const int64_t n = T.n, cap = T.node_cap, cap_c = W.cap_c;
    hipError_t e = launch_morton_order(t, x, s);
    if (e != hipSuccess)
        return e;
    const int gs = (int)std::min<int64_t>((n + 255) / 256, 2048);
    // cells of even levels lie in the first buffer, of odd levels in the second
    uint32_t *Q[2] = {W.q, W.q_tmp};
    int32_t *perm[2] = {W.perm_tmp, W.perm_tmp + n};
    k_com_zero<<<1, COM_CTL, 0, s>>>(W.ctl);
    if (m)
        k_com_mmax<<<std::min(gs, 256), 256, 0, s>>>(m, n, W.ctl);
    k_com_init<<<gs, 256, 0, s>>>(x, m, n, t.bbox, W.ctl, t.vals0, perm[0], Q[0]);
    k_com_root<<<1, 256, 0, s>>>(n, W.node, cap, W.act[0], W.act_choff[0], W.chk[0], cap_c, W.ren,
                                 W.ctl);
    // levels that a balanced tree has above the finished cells, and one more
    int batch = n > COM_SUB ? 1 : 0;
    while (batch && (n >> batch) > COM_SUB)
        ++batch;
    batch = batch ? batch + 1 : 0;
    int level = 0;
    do {
        for (; batch > 0; --batch, ++level) {
            const int cur = level & 1;
            const int64_t acts =
                std::min<int64_t>(level < 30 ? 1ll << level : W.cap_a, com_max_active(n));
            const int C = (int)std::min<int64_t>(n / COM_CHUNK + acts, cap_c);
            k_com_stats<<<C, CB, 0, s>>>(Q[cur], n, W.chk[cur], cap_c, W.cpart, W.ctl);
            k_com_count<<<C, CB, 0, s>>>(Q[cur], n, W.chk[cur], cap_c, W.act[cur],
                                         W.act_choff[cur], W.node, cap, W.cpart, W.split, W.cleft,
                                         W.ctl);
            k_com_scatter<<<C, CB, 0, s>>>(Q[cur], perm[cur], n, W.chk[cur], cap_c, W.act[cur],
                                           W.act_choff[cur], W.node, cap, W.split, W.cleft,
                                           Q[cur ^ 1], perm[cur ^ 1], W.ctl);
            k_com_next<<<1, NEXT_T, 0, s>>>(level, W.node, cap, W.act[cur ^ 1],
                                            W.act_choff[cur ^ 1], W.chk[cur ^ 1], cap_c, W.ren,
                                            W.ctl);
        }
        if ((e = read_ctl(t, s)) != hipSuccess)
            return e;
        batch = 1;
    } while (W.h_ctl[CA] > 0);
    const int nfin = (int)W.h_ctl[CS], ntop = (int)W.h_ctl[CNN];
    k_com_finish<<<nfin, FIN_T, 0, s>>>(Q[0], perm[0], Q[1], perm[1], n, W.node, cap, T.leaf_size,
                                        W.ren, W.rec, t.perm, W.ctl);
    k_com_number<<<1, 1024, 0, s>>>(W.node, cap, W.ren, W.ctl);
    uint32_t *key = (uint32_t *)t.keys0, *val = (uint32_t *)t.keys1;
    const ComOut O = {t.first, t.count, t.left, t.right, t.parent, t.level, t.axis, t.node_leaf,
                      t.leaf_node, t.big_nodes, key, val};
    const int top_blocks = std::min((ntop + 255) / 256, 256);
    k_com_emit<<<nfin + top_blocks, 256, 0, s>>>(nfin, W.node, cap, W.ren, W.rec, O, W.ctl);
    if ((e = read_ctl(t, s)) != hipSuccess)
        return e;
    T.nnodes = (int)W.h_ctl[CTOT];
    T.nleaves = (int)W.h_ctl[CLEAF];
    T.depth = (int)W.h_ctl[CDEP];
    T.nbig = (int)W.h_ctl[CNBIG];
    T.lvl_int_off.assign(1, 0);
    for (int l = 0; l < T.depth && l < COM_MAX_DEPTH; ++l)
        T.lvl_int_off.push_back(T.lvl_int_off.back() + (int)W.h_ctl[CLVL + l]);
    return radix_sort_u32(key, val, key + cap, (uint32_t *)t.int_nodes, T.nnodes, 1, 1, t.rs_hist,
                          t.rs_tot, s, 8);
}

}  // namespace fmm
