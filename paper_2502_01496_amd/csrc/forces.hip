// Far and near field on gfx950.
//
// M2L (eq. (6) of the paper and its first two r-derivatives): for a sink cell
// and a source cell with mass M, quadrupole Q about its centre of mass, and
// r = c_sink - c_source, the local expansion is L = (a, grad a, grad grad a)
// at c_sink.  With g_n = (-1)^n (2n-1)!! r^-(2n+1) (so d/dr_i g_n = g_{n+1} r_i),
// q = Q r, qq = r.q and
//   a0 = M g1 + g3 qq / 6,  a1 = M g2 + g4 qq / 6,  a2 = M g3 + g5 qq / 6,
//   b2 = g2 / 3, b3 = g3 / 3, b4 = g4 / 3:
//   L1_i   = a0 r_i + b2 q_i                                   (= eq. (6))
//   L2_ij  = a1 r_i r_j + a0 d_ij + b3 (r_i q_j + q_i r_j) + b2 Q_ij
//   L3_ijk = a2 r_i r_j r_k + a1 (d_ij r_k + d_ik r_j + d_jk r_i)
//            + b4 (r_i r_j q_k + r_i r_k q_j + r_j r_k q_i)
//            + b3 (d_ij q_k + d_ik q_j + d_jk q_i) + b3 (r_i Q_jk + r_j Q_ik + r_k Q_ij)
// The second expansion form (eqs. (25)-(26) with p = 3: combined order of the
// source and sink offsets at most 2) keeps L1 and replaces L2, L3 by the
// derivatives of the monopole field alone:
//   L2_ij  = A1 r_i r_j + A0 d_ij,  L3_ijk = A2 r_i r_j r_k + A1 (d_ij r_k + d_ik r_j + d_jk r_i),
//   A0 = M g1, A1 = M g2, A2 = M g3 (highest power of 1/r: 4, against 6).
// L2P (eq. (8)): a(y) = L1 + L2 y + 1/2 L3 : y y, y = x - c_sink.
// Near field (Sec. 3, eqs. (12)-(15), M4 kernel, R_kern = 2): particle i gets
//   -m_j * 1/2 [g(r, h_i) + g(r, h_j)] * (x_i - x_j) from every j != i of its
// near cells, with g = phi'/r:
//   q < 1:      h^-3 (4/3 - 6/5 q^2 + 1/2 q^3)
//   1 <= q < 2: h^-3 (8/3 - 3 q + 6/5 q^2 - 1/6 q^3) - 1/(15 r^3)
//   q >= 2:     1/r^3.
//
// Storage: symmetric rank-2 (xx,xy,xz,yy,yz,zz); rank-3
// (xxx,xxy,xxz,xyy,xyz,xzz,yyy,yyz,yzz,zzz).
#include <type_traits>

#include "fmm_internal.h"

namespace fmm {

template <typename T>
__device__ __forceinline__ T rsqrt_t(T x);
template <>
__device__ __forceinline__ double rsqrt_t<double>(double x) { return rsqrt(x); }
template <>
__device__ __forceinline__ float rsqrt_t<float>(float x) { return rsqrtf(x); }

// Second expansion form: L1 as eq. (6), L2 and L3 from the monopole only.
template <typename T>
__device__ __forceinline__ void m2l_acc_dehnen(T rx, T ry, T rz, T M, const T *Q, T *L)
{
    const T r2 = rx * rx + ry * ry + rz * rz;
    const T u = rsqrt_t<T>(r2);
    const T u2 = u * u;
    const T g1 = -u * u2;
    const T g2 = T(-3) * g1 * u2;
    const T g3 = T(-5) * g2 * u2;
    const T Qxx = Q[0], Qxy = Q[1], Qxz = Q[2], Qyy = Q[3], Qyz = Q[4], Qzz = Q[5];
    const T qx = Qxx * rx + Qxy * ry + Qxz * rz;
    const T qy = Qxy * rx + Qyy * ry + Qyz * rz;
    const T qz = Qxz * rx + Qyz * ry + Qzz * rz;
    const T qq = qx * rx + qy * ry + qz * rz;
    const T sixth = T(1) / T(6), third = T(1) / T(3);
    const T a0 = M * g1 + g3 * qq * sixth;
    const T b2 = g2 * third;
    const T A0 = M * g1, A1 = M * g2, A2 = M * g3;
    L[0] += a0 * rx + b2 * qx;
    L[1] += a0 * ry + b2 * qy;
    L[2] += a0 * rz + b2 * qz;
    const T A1x = A1 * rx, A1y = A1 * ry, A1z = A1 * rz;
    L[3] += A1x * rx + A0;
    L[4] += A1x * ry;
    L[5] += A1x * rz;
    L[6] += A1y * ry + A0;
    L[7] += A1y * rz;
    L[8] += A1z * rz + A0;
    const T A2x = A2 * rx, A2y = A2 * ry, A2z = A2 * rz;
    L[9] += A2x * rx * rx + T(3) * A1x;
    L[10] += A2x * rx * ry + A1y;
    L[11] += A2x * rx * rz + A1z;
    L[12] += A2x * ry * ry + A1x;
    L[13] += A2x * ry * rz;
    L[14] += A2x * rz * rz + A1x;
    L[15] += A2y * ry * ry + T(3) * A1y;
    L[16] += A2y * ry * rz + A1z;
    L[17] += A2y * rz * rz + A1y;
    L[18] += A2z * rz * rz + T(3) * A1z;
}

// One source -> sink M2L, accumulated into L[19]; FORM is FMM_EXPANSION_*.
template <typename T, int FORM>
__device__ __forceinline__ void m2l_acc(T rx, T ry, T rz, T M, const T *Q, T *L)
{
    if constexpr (FORM == FMM_EXPANSION_DEHNEN) {
        m2l_acc_dehnen<T>(rx, ry, rz, M, Q, L);
        return;
    }
    const T r2 = rx * rx + ry * ry + rz * rz;
    const T u = rsqrt_t<T>(r2);
    const T u2 = u * u;
    const T g1 = -u * u2;
    const T g2 = T(-3) * g1 * u2;
    const T g3 = T(-5) * g2 * u2;
    const T g4 = T(-7) * g3 * u2;
    const T g5 = T(-9) * g4 * u2;
    const T Qxx = Q[0], Qxy = Q[1], Qxz = Q[2], Qyy = Q[3], Qyz = Q[4], Qzz = Q[5];
    const T qx = Qxx * rx + Qxy * ry + Qxz * rz;
    const T qy = Qxy * rx + Qyy * ry + Qyz * rz;
    const T qz = Qxz * rx + Qyz * ry + Qzz * rz;
    const T qq = qx * rx + qy * ry + qz * rz;
    const T sixth = T(1) / T(6), third = T(1) / T(3);
    const T a0 = M * g1 + g3 * qq * sixth;
    const T a1 = M * g2 + g4 * qq * sixth;
    const T a2 = M * g3 + g5 * qq * sixth;
    const T b2 = g2 * third, b3 = g3 * third, b4 = g4 * third;
    // L1
    L[0] += a0 * rx + b2 * qx;
    L[1] += a0 * ry + b2 * qy;
    L[2] += a0 * rz + b2 * qz;
    // L2
    L[3] += a1 * rx * rx + a0 + b3 * (T(2) * rx * qx) + b2 * Qxx;
    L[4] += a1 * rx * ry + b3 * (rx * qy + qx * ry) + b2 * Qxy;
    L[5] += a1 * rx * rz + b3 * (rx * qz + qx * rz) + b2 * Qxz;
    L[6] += a1 * ry * ry + a0 + b3 * (T(2) * ry * qy) + b2 * Qyy;
    L[7] += a1 * ry * rz + b3 * (ry * qz + qy * rz) + b2 * Qyz;
    L[8] += a1 * rz * rz + a0 + b3 * (T(2) * rz * qz) + b2 * Qzz;
    // L3: the delta terms are folded per component
    const T a2x = a2 * rx, a2y = a2 * ry, a2z = a2 * rz;
    // xxx: rrr = x^3; dr = 3x; rrq = 3 x^2 qx; dq = 3 qx; rQ = 3 x Qxx
    L[9] += a2x * rx * rx + a1 * T(3) * rx + b4 * (T(3) * rx * rx * qx) + b3 * (T(3) * qx) +
            b3 * (T(3) * rx * Qxx);
    // xxy: dr = y; rrq = x^2 qy + 2 x y qx; dq = qy; rQ = 2 x Qxy + y Qxx
    L[10] += a2x * rx * ry + a1 * ry + b4 * (rx * rx * qy + T(2) * rx * ry * qx) + b3 * qy +
             b3 * (T(2) * rx * Qxy + ry * Qxx);
    // xxz
    L[11] += a2x * rx * rz + a1 * rz + b4 * (rx * rx * qz + T(2) * rx * rz * qx) + b3 * qz +
             b3 * (T(2) * rx * Qxz + rz * Qxx);
    // xyy: dr = x; rrq = y^2 qx + 2 x y qy; dq = qx; rQ = x Qyy + 2 y Qxy
    L[12] += a2x * ry * ry + a1 * rx + b4 * (ry * ry * qx + T(2) * rx * ry * qy) + b3 * qx +
             b3 * (rx * Qyy + T(2) * ry * Qxy);
    // xyz: dr = 0; rrq = xy qz + xz qy + yz qx; dq = 0; rQ = x Qyz + y Qxz + z Qxy
    L[13] += a2x * ry * rz + b4 * (rx * ry * qz + rx * rz * qy + ry * rz * qx) +
             b3 * (rx * Qyz + ry * Qxz + rz * Qxy);
    // xzz
    L[14] += a2x * rz * rz + a1 * rx + b4 * (rz * rz * qx + T(2) * rx * rz * qz) + b3 * qx +
             b3 * (rx * Qzz + T(2) * rz * Qxz);
    // yyy
    L[15] += a2y * ry * ry + a1 * T(3) * ry + b4 * (T(3) * ry * ry * qy) + b3 * (T(3) * qy) +
             b3 * (T(3) * ry * Qyy);
    // yyz
    L[16] += a2y * ry * rz + a1 * rz + b4 * (ry * ry * qz + T(2) * ry * rz * qy) + b3 * qz +
             b3 * (T(2) * ry * Qyz + rz * Qyy);
    // yzz
    L[17] += a2y * rz * rz + a1 * ry + b4 * (rz * rz * qy + T(2) * ry * rz * qz) + b3 * qy +
             b3 * (ry * Qzz + T(2) * rz * Qyz);
    // zzz
    L[18] += a2z * rz * rz + a1 * T(3) * rz + b4 * (T(3) * rz * rz * qz) + b3 * (T(3) * qz) +
             b3 * (T(3) * rz * Qzz);
}

// FP64 sums of eq. (6)'s form over the sources of one lane, in another
// grouping of the same terms: with v_n = r^-(2n+1), t = 35/2 v4 q + a2/6 r,
// P_ij = r_i t_j + t_i r_j + b3 Q_ij and s = a1/2 r + b3 q,
//   L2_ij  = r_i s_j + s_i r_j + b2 Q_ij + a0 d_ij,
//   L3_ijk = r_i P_jk + r_j P_ik + r_k P_ij + d_ij w_k + d_ik w_j + d_jk w_i,
//   w = s + a1/2 r,
// and the terms with d_ij (a0 and w) are summed apart and added at the end:
// 120 FP64 instructions per source instead of 190.  With the source's record
// read part by part (an L1 lookup per lane and 16 bytes, 5.2 per source, which
// bounded the leaf M2L) they gave 218 -> 205 us (binary, 2^19 particles) and
// 2.09 -> 2.00 ms (clumpy cube, 2^22), with the gather by quads (2 lookups per
// source) 181 us and 1.63 ms.  The plain FP64 sums (1.66 -> 1.85 ms for Plummer,
// 2^19) and the FP32 form (164 -> 169 us, binary) are not faster with it: they
// are bound by their arithmetic, and the parts in flight cost a wavefront.
struct M2lSum64 {
    double l1[3], l2[6], l3[10], a0, w[3];
    __device__ __forceinline__ void clear()
    {
#pragma unroll
        for (int k = 0; k < 3; ++k)
            l1[k] = w[k] = 0.0;
#pragma unroll
        for (int k = 0; k < 6; ++k)
            l2[k] = 0.0;
#pragma unroll
        for (int k = 0; k < 10; ++k)
            l3[k] = 0.0;
        a0 = 0.0;
    }
    __device__ __forceinline__ void add(double x, double y, double z, double M, const double *Q)
    {
        const double u = rsqrt_pos(x * x + y * y + z * z);  // r > 0: far cells are apart
        const double u2 = u * u;
        const double v1 = u * u2, v2 = v1 * u2, v3 = v2 * u2, v4 = v3 * u2, v5 = v4 * u2;
        const double qx = Q[0] * x + Q[1] * y + Q[2] * z;
        const double qy = Q[1] * x + Q[3] * y + Q[4] * z;
        const double qz = Q[2] * x + Q[4] * y + Q[5] * z;
        const double qq = 2.5 * (qx * x + qy * y + qz * z);
        const double m0 = M * v1 + qq * v3;                             // -a0
        const double h1 = (1.5 * M) * v2 + (3.5 * qq) * v4;             // a1 / 2
        const double c2 = -((2.5 * M) * v3 + (10.5 * qq) * v5);         // a2 / 6
        const double b3 = -5.0 * v3, c4 = 17.5 * v4;
        const double tx = c4 * qx + c2 * x, ty = c4 * qy + c2 * y, tz = c4 * qz + c2 * z;
        const double sx = b3 * qx + h1 * x, sy = b3 * qy + h1 * y, sz = b3 * qz + h1 * z;
        const double x2 = x + x, y2 = y + y, z2 = z + z;
        l1[0] += v2 * qx - m0 * x;
        l1[1] += v2 * qy - m0 * y;
        l1[2] += v2 * qz - m0 * z;
        a0 -= m0;
        l2[0] = fma(v2, Q[0], fma(x2, sx, l2[0]));
        l2[1] = fma(v2, Q[1], fma(y, sx, fma(x, sy, l2[1])));
        l2[2] = fma(v2, Q[2], fma(z, sx, fma(x, sz, l2[2])));
        l2[3] = fma(v2, Q[3], fma(y2, sy, l2[3]));
        l2[4] = fma(v2, Q[4], fma(z, sy, fma(y, sz, l2[4])));
        l2[5] = fma(v2, Q[5], fma(z2, sz, l2[5]));
        w[0] = fma(h1, x, w[0] + sx);
        w[1] = fma(h1, y, w[1] + sy);
        w[2] = fma(h1, z, w[2] + sz);
        const double pxx = fma(x2, tx, b3 * Q[0]), pyy = fma(y2, ty, b3 * Q[3]),
                     pzz = fma(z2, tz, b3 * Q[5]);
        const double pxy = fma(x, ty, fma(y, tx, b3 * Q[1])),
                     pxz = fma(x, tz, fma(z, tx, b3 * Q[2])),
                     pyz = fma(y, tz, fma(z, ty, b3 * Q[4]));
        l3[0] = fma(x, pxx, l3[0]);
        l3[1] = fma(x2, pxy, fma(y, pxx, l3[1]));
        l3[2] = fma(x2, pxz, fma(z, pxx, l3[2]));
        l3[3] = fma(y2, pxy, fma(x, pyy, l3[3]));
        l3[4] = fma(x, pyz, fma(y, pxz, fma(z, pxy, l3[4])));
        l3[5] = fma(z2, pxz, fma(x, pzz, l3[5]));
        l3[6] = fma(y, pyy, l3[6]);
        l3[7] = fma(y2, pyz, fma(z, pyy, l3[7]));
        l3[8] = fma(z2, pyz, fma(y, pzz, l3[8]));
        l3[9] = fma(z, pzz, l3[9]);
    }
    __device__ __forceinline__ void total(double *L) const
    {
        L[0] = l1[0];
        L[1] = l1[1];
        L[2] = l1[2];
        L[3] = l2[0] + a0;
        L[4] = l2[1];
        L[5] = l2[2];
        L[6] = l2[3] + a0;
        L[7] = l2[4];
        L[8] = l2[5] + a0;
        L[9] = 3.0 * (l3[0] + w[0]);
        L[10] = l3[1] + w[1];
        L[11] = l3[2] + w[2];
        L[12] = l3[3] + w[0];
        L[13] = l3[4];
        L[14] = l3[5] + w[0];
        L[15] = 3.0 * (l3[6] + w[1]);
        L[16] = l3[7] + w[2];
        L[17] = l3[8] + w[1];
        L[18] = 3.0 * (l3[9] + w[2]);
    }
};

// ---------------------------------------------------------------- list pieces
// Pieces per leaf for a list of min(cnt, cap) entries of `mult` work units
// each: ceil(work / per), at least one.
__global__ void k_piece_count(const int32_t *__restrict__ cnt, int cap, int nleaves, int mult,
                              int64_t per, int32_t *np)
{
    const int lf = blockIdx.x * blockDim.x + threadIdx.x;
    if (lf >= nleaves)
        return;
    const int64_t wk = (int64_t)max(0, min(cnt[lf], cap)) * mult;
    np[lf] = (int32_t)max<int64_t>(1, (wk + per - 1) / per);
}

__global__ void k_piece_fill(const int64_t *__restrict__ off, const int32_t *__restrict__ np,
                             int nleaves, int2 *list)
{
    const int lf = blockIdx.x * blockDim.x + threadIdx.x;
    if (lf >= nleaves)
        return;
    const int64_t extra = off[nleaves] - nleaves;
    for (int k = 0; k < np[lf]; ++k)
        list[piece_pos(off, extra, lf, k)] = make_int2(lf, k);
}

// Folding the partial sums of a split leaf's pieces, in piece order: one
// thread per extra list entry, the one holding piece 1 of its leaf folds it.
template <typename T>
__global__ __launch_bounds__(256) void k_m2l_fold(const int32_t *__restrict__ leaf_node,
                                                  const int64_t *__restrict__ off,
                                                  const int2 *__restrict__ list, int extra,
                                                  const T *__restrict__ part, T *Lout)
{
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= extra || list[e].y != 1)
        return;
    const int lf = list[e].x;
    T L[19];
#pragma unroll
    for (int k = 0; k < 19; ++k)
        L[k] = T(0);
    const int np = (int)(off[lf + 1] - off[lf]);
    for (int q = 0; q < np; ++q) {
        const T *pp = part + (int64_t)NLOC * piece_pos(off, extra, lf, q);
#pragma unroll
        for (int k = 0; k < 19; ++k)
            L[k] += pp[k];
    }
    T *o = Lout + (int64_t)NLOC * leaf_node[lf];
#pragma unroll
    for (int k = 0; k < 19; ++k)
        o[k] = L[k];
    o[19] = T(0);
}

// ---------------------------------------------------------------- M2L at the leaves
// The FP32 form with the load of the source record apart from the
// arithmetic, so that the next source's record can be in flight while the
// current one is evaluated.
struct M2lSrc32 {
    double4 cb;
    float4 f0, f1;
};
__device__ __forceinline__ void m2l_src_load(const double *__restrict__ recA,
                                             const float *__restrict__ recF, int b, M2lSrc32 &S)
{
    S.cb = *(const double4 *)(recA + (int64_t)NREC * b);
    S.f0 = *(const float4 *)(recF + (int64_t)NREC * b);
    S.f1 = *(const float4 *)(recF + (int64_t)NREC * b + 4);
}
template <int FORM>
__device__ __forceinline__ void m2l_src_eval(const M2lSrc32 &S, double c0, double c1, double c2,
                                             float *L)
{
    const float Q[6] = {S.f0.y, S.f0.z, S.f0.w, S.f1.x, S.f1.y, S.f1.z};
    m2l_acc<float, FORM>((float)(c0 - S.cb.x), (float)(c1 - S.cb.y), (float)(c2 - S.cb.z), S.f0.x,
                         Q, L);
}

// M2L of eq. (6) at the sink leaves.  8 lanes per unit, 8 units per wave
// (consecutive leaves, whose far lists largely coincide, so the wave's loads
// of a source record often share an address); lanes stride the far list,
// and a butterfly sum over the unit's lanes ends each
// piece of `per` list entries; piece sums add up in piece order, starting
// from zero (fixed order: deterministic).  A unit is a leaf (pieces == nullptr: all its pieces in
// turn, total to Lout) or one entry of the piece list: the only piece of its
// leaf (total to Lout) or one piece of a split list (its sum to part, added
// by k_m2l_fold), with bit-identical totals either way.
constexpr int M2L_LANES = 8;  // lanes per unit

// REGROUP: FP64 sums in the grouping of M2lSum64 (eq. (6)'s form).  The FP64
// expansions that the reverse pass of FP32 trees forms keep the plain order, so
// that its results, rounded to FP32, stay the same to the bit; that is a choice,
// at 1.95 against 1.56 ms (clumpy cube, 2^22).
template <typename T, int FORM, bool REGROUP>
__global__ __launch_bounds__(256) void k_m2l_leaf(
    const double *__restrict__ recA, const double *__restrict__ recQ,
    const float *__restrict__ recF, const int32_t *__restrict__ leaf_node, int nunits,
    const int32_t *__restrict__ far_cnt, const int32_t *__restrict__ far_src, int cap_far,
    T *Lout, const int2 *__restrict__ pieces, int per, T *part)
{
    const int g = (xcd_block(blockIdx.x, gridDim.x) * 256 + threadIdx.x) / M2L_LANES;
    const int sub = threadIdx.x & (M2L_LANES - 1);
    const bool valid = g < nunits;
    const int2 pc = pieces && valid ? pieces[g] : make_int2(valid ? g : 0, 0);
    const int lf = pc.x;
    const int v = valid ? leaf_node[lf] : 0;
    const double *rv = recA + (int64_t)NREC * v;
    const double c0 = rv[0], c1 = rv[1], c2 = rv[2];
    const int nfull = valid ? max(0, min(far_cnt[lf], cap_far)) : 0;
    const int lo = pieces ? pc.y * per : 0;
    const int hi = pieces ? min(nfull, lo + per) : nfull;
    const int32_t *fl = far_src + (int64_t)lf * cap_far;
    const bool split = pieces && nfull > per;
    T *o = split ? part + (int64_t)NLOC * g : Lout + (int64_t)NLOC * v;
    if (valid && sub == 0) {
#pragma unroll
        for (int k = 0; k < NLOC; ++k)
            o[k] = T(0);
    }
    for (int p0 = lo; p0 < hi; p0 += per) {
        const int p1 = min(hi, p0 + per);
        T L[19];
#pragma unroll
        for (int k = 0; k < 19; ++k)
            L[k] = T(0);
        if constexpr (std::is_same<T, float>::value) {
            // FP32: the next source's record and the index after it are in
            // flight while the current source is evaluated (the FP64 form
            // keeps one wavefront more per SIMD without them, which pays more)
            M2lSrc32 cur;
            int bn = 0;
            if (p0 + sub < p1) {
                m2l_src_load(recA, recF, fl[p0 + sub], cur);
                if (p0 + sub + M2L_LANES < p1)
                    bn = fl[p0 + sub + M2L_LANES];
            }
            for (int k = p0 + sub; k < p1; k += M2L_LANES) {
                M2lSrc32 nxt;
                if (k + M2L_LANES < p1) {
                    m2l_src_load(recA, recF, bn, nxt);
                    if (k + 2 * M2L_LANES < p1)
                        bn = fl[k + 2 * M2L_LANES];
                }
                m2l_src_eval<FORM>(cur, c0, c1, c2, L);
                cur = nxt;
            }
        } else if constexpr (REGROUP) {
            // the next source's record and the index after it are in flight.
            // All lanes of a unit stay in the loop (the gather needs whole
            // quads): a lane past the piece's end reads the root's record and
            // adds nothing
            M2lSum64 S;
            S.clear();
            const double2 *A2 = (const double2 *)recA;
            const int b0 = p0 + sub < p1 ? fl[p0 + sub] : 0;
            QuadRecord rec;
            rec.fetch(recQ, b0);
            double2 cn = A2[NREC / 2 * (int64_t)b0];
            int bn = p0 + sub + M2L_LANES < p1 ? fl[p0 + sub + M2L_LANES] : 0;
            for (int k0 = p0; k0 < p1; k0 += M2L_LANES) {
                int4 i0, i1, i2, i3;
                rec.parts(i0, i1, i2, i3);
                const double2 cxy = cn;
                if (k0 + M2L_LANES < p1) {
                    rec.fetch(recQ, bn);
                    cn = A2[NREC / 2 * (int64_t)bn];
                    bn = k0 + sub + 2 * M2L_LANES < p1 ? fl[k0 + sub + 2 * M2L_LANES] : 0;
                }
                const double2 q01 = as_double2(i0), q23 = as_double2(i1), q45 = as_double2(i2),
                              czm = as_double2(i3);
                const double Q[6] = {q01.x, q01.y, q23.x, q23.y, q45.x, q45.y};
                if (k0 + sub < p1)
                    S.add(c0 - cxy.x, c1 - cxy.y, c2 - czm.x, czm.y, Q);
            }
            S.total(L);
        } else {
            // the next source's index is loaded one interaction ahead
            int bn = p0 + sub < p1 ? fl[p0 + sub] : 0;
            for (int k = p0 + sub; k < p1; k += M2L_LANES) {
                const int b = bn;
                if (k + M2L_LANES < p1)
                    bn = fl[k + M2L_LANES];
                const double4 cb = *(const double4 *)(recA + (int64_t)NREC * b);
                const double *qb = recQ + (int64_t)NREC * b;
                const double2 q01 = *(const double2 *)qb, q23 = *(const double2 *)(qb + 2),
                              q45 = *(const double2 *)(qb + 4);
                const double Q[6] = {q01.x, q01.y, q23.x, q23.y, q45.x, q45.y};
                m2l_acc<double, FORM>(c0 - cb.x, c1 - cb.y, c2 - cb.z, cb.w, Q, L);
            }
        }
#pragma unroll
        for (int off = M2L_LANES / 2; off >= 1; off >>= 1)
#pragma unroll
            for (int k = 0; k < 19; ++k)
                L[k] += __shfl_xor(L[k], off);
        // the piece sums add up in the output itself (no registers held for a
        // running total), in piece order: 0 + L_0 + L_1 + ...
        if (valid && sub == 0) {
#pragma unroll
            for (int k = 0; k < 19; ++k)
                o[k] = o[k] + L[k];
        }
    }
}

// ---------------------------------------------------------------- P2P + L2P, FP64 (mutual walk)
__device__ __forceinline__ double m4g_f64(double q, double hinv3, double u3)
{
    // both pieces are evaluated and selected (no divergent branches)
    const double p1 = hinv3 * (4.0 / 3.0 + q * q * (-1.2 + 0.5 * q));
    const double p2 = hinv3 * (8.0 / 3.0 + q * (-3.0 + q * (1.2 - q * (1.0 / 6.0)))) -
                      u3 * (1.0 / 15.0);
    const double g = __builtin_unpredictable(q < 2.0) ? p2 : u3;
    return __builtin_unpredictable(q < 1.0) ? p1 : g;
}

// m / r^3 for finite r2 > 0: the hardware reciprocal square root y refined
// once with the series (1 - e)^(-1/2) = 1 + e/2 + 3/8 e^2 + O(e^3),
// e = 1 - r2 y^2, then cubed.
__device__ __forceinline__ double m_over_r3(double r2, double m)
{
    const double y = __builtin_amdgcn_rsq(r2);
    const double e = fma(-(r2 * y), y, 1.0);
    const double u = fma(y * e, fma(e, 0.375, 0.5), y);
    return m * ((u * u) * u);
}

// Reduce-scatter of 24 per-lane values over the 64 lanes of a wavefront.
// Each xor step halves the set of values a lane keeps (it sends the other
// half to its partner); after the steps over lane bits 5..1 a lane holds the
// partial sum of one value, and a last butterfly step finishes it.  Value
// index held by lane l: 12 b5 + 6 b4 + 3 b3 + (2 b2 + b1), valid when
// (2 b2 + b1) < 3.
template <typename T>
__device__ __forceinline__ T xchg_keep(T keep, T send, int off)
{
    return keep + __shfl_xor(send, off);
}

// Value index a lane holds after reduce_scatter24 (-1: none).
__device__ __forceinline__ int rs24_index(int lane)
{
    const int sub = 2 * ((lane >> 2) & 1) + ((lane >> 1) & 1);
    return sub < 3 ? 12 * ((lane >> 5) & 1) + 6 * ((lane >> 4) & 1) + 3 * ((lane >> 3) & 1) + sub
                   : -1;
}

template <typename T>
__device__ __forceinline__ T reduce_scatter24(const T *v, int lane)
{
    const bool b5 = lane & 32, b4 = lane & 16, b3 = lane & 8, b2 = lane & 4, b1 = lane & 2;
    T a[12];
#pragma unroll
    for (int k = 0; k < 12; ++k)
        a[k] = xchg_keep<T>(b5 ? v[12 + k] : v[k], b5 ? v[k] : v[12 + k], 32);
    T b[6];
#pragma unroll
    for (int k = 0; k < 6; ++k)
        b[k] = xchg_keep<T>(b4 ? a[6 + k] : a[k], b4 ? a[k] : a[6 + k], 16);
    T cc[3];
#pragma unroll
    for (int k = 0; k < 3; ++k)
        cc[k] = xchg_keep<T>(b3 ? b[3 + k] : b[k], b3 ? b[k] : b[3 + k], 8);
    const T d0 = xchg_keep<T>(b2 ? cc[2] : cc[0], b2 ? cc[0] : cc[2], 4);
    const T d1 = xchg_keep<T>(b2 ? T(0) : cc[1], b2 ? cc[1] : T(0), 4);
    T e = xchg_keep<T>(b1 ? d1 : d0, b1 ? d0 : d1, 2);
    e += __shfl_xor(e, 1);
    return e;
}

// Near field of the mutual walk's lists.  One wavefront per sink leaf; P2P_NS
// sink particles per pass are wave-uniform (with SKIP, for trees whose leaves
// are not all full, absent ones are branched over: without absent ones the
// branches cost 2 to 4 %), and a step takes 8 source blocks (a near leaf gives
// ceil(leaf_size / 8) blocks of at most 8 particles): lane = 8 g + t holds
// particle t of the g-th block, loaded once per pass.  The block ranges of
// a chunk of the near list are staged in LDS (empty blocks dropped), and the
// next step's sources load while the current step computes.  Missing
// sources are the null record (far away, zero mass, zero smoothing length),
// which adds exactly zero.
//
// Every pair is first tested against the softening support of eqs. (14)-(15),
// with the largest 4 h^2 of the pass's sinks standing in for the sink's own:
// r^2 < max(H4, 4 h_j^2).  Pairs outside it are Newtonian for certain and
// take the form m / r^3 in the step.  Pairs inside are appended to their
// sink's queue in LDS (the source's tree position) and evaluated with the M4
// kernel, which is exact on both sides of the support, 64 at a time, so that
// the softened form runs with every lane busy instead of stalling a whole
// step whenever one of its pairs may be softened (a queue is drained each
// time it has gathered 64 pairs, and at the end of the pass).  The order of
// all additions depends on the lists only, so results are bitwise
// reproducible.
// The per-lane sums are reduce-scattered so that the lane holding component
// c of sink s adds L2P and writes G * a.
// One wavefront per workgroup: the leaves' near lists differ in length, and a
// workgroup's slots are only freed when its last wavefront ends.
constexpr int P2P_WAVES = 1;
constexpr int P2P_WG = 64 * P2P_WAVES;
constexpr int P2P_NS = 8;        // sinks per pass
constexpr int P2P_QCAP = 128;    // softened pairs a sink's queue holds (a step adds <= 64)
constexpr int P2P_BLOCKS = 256;  // source blocks staged in LDS per chunk

// Stage the non-empty blocks of list entries [c0, c0 + nc) (entry k: block
// k % nsub of near leaf k / nsub) in list order; returns their number.
__device__ __forceinline__ int stage_blocks_in_order(const int32_t *__restrict__ nl, int c0, int nc,
                                                     int nsub, const int32_t *__restrict__ first,
                                                     const int32_t *__restrict__ count, int lane,
                                                     int2 *R)
{
    int ne = 0;
    for (int k0 = 0; k0 < nc; k0 += 64) {
        const int k = k0 + lane;
        int2 r = make_int2(0, 0);
        if (k < nc) {
            const int e = (c0 + k) / nsub, u = (c0 + k) - e * nsub;
            const int bn = nl[e];
            r = make_int2(first[bn] + 8 * u, max(0, min(8, count[bn] - 8 * u)));
        }
        const bool keep = r.y > 0;
        const uint64_t mk = __ballot(keep);
        if (keep)
            R[ne + __popcll(mk & lanemask_lt())] = r;
        ne += __popcll(mk);
    }
    if (lane < 8)
        R[ne + lane] = make_int2(0, 0);  // eight empty blocks after the last one
    return ne;
}

// Source particle of a lane in block rg (the null record past its end).
__device__ __forceinline__ int64_t block_src(int2 rg, int slot, int64_t nnull)
{
    return slot < rg.y ? (int64_t)rg.x + slot : nnull;
}

// The softened pairs of sink q: cnt <= 64 entries of its queue from position
// head, one per lane, with the mean of the two M4 kernels.
template <int NS>
__device__ __forceinline__ void p2p_drain_f64(const double4 *__restrict__ pm,
                                              const double4 *__restrict__ ph,
                                              const int32_t *Q, int head, int cnt, int lane,
                                              int64_t nnull, double sx, double sy, double sz,
                                              double shi, double sh3, double &ax, double &ay,
                                              double &az)
{
    const int64_t j = lane < cnt ? (int64_t)Q[(head + lane) & (P2P_QCAP - 1)] : nnull;
    const double4 xj = pm[j];
    const double4 hj = ph[j];
    const double dx = sx - xj.x, dy = sy - xj.y, dz = sz - xj.z;
    const double r2 = dx * dx + dy * dy + dz * dz;
    const double u = r2 > 0.0 ? rsqrt_pos(r2) : 0.0;
    const double r = r2 * u;
    const double u3 = u * u * u;
    const double gi = m4g_f64(r * shi, sh3, u3);
    const double gj = m4g_f64(r * hj.x, hj.y, u3);
    const double fm = 0.5 * xj.w * (gi + gj);
    ax -= fm * dx;
    ay -= fm * dy;
    az -= fm * dz;
}

template <bool SKIP>
__global__ __launch_bounds__(P2P_WG) __attribute__((amdgpu_waves_per_eu(4, 8))) void k_p2p_src_f64(
    const double4 *__restrict__ pm, const double4 *__restrict__ ph,
    const int32_t *__restrict__ first, const int32_t *__restrict__ count,
    const int32_t *__restrict__ leaf_node, int nleaves, const int32_t *__restrict__ near_cnt,
    const int32_t *__restrict__ near_src, int cap_near, int nsub, const double *__restrict__ Lloc,
    const double *__restrict__ recA, const int32_t *__restrict__ perm, double G, double r_kern,
    int64_t nnull, double *aout, const int2 *__restrict__ pieces, int per, double *part,
    int part_stride)
{
    constexpr int NS = P2P_NS;
    __shared__ int2 rng[P2P_WAVES][P2P_BLOCKS + 8];
    __shared__ int32_t que[P2P_WAVES][NS][P2P_QCAP];
    __shared__ double2 shh[P2P_WAVES][NS];  // 1/h, 1/h^3 of the pass's sinks
    (void)r_kern;
    const int w = threadIdx.x >> 6;
    const int unit =
        __builtin_amdgcn_readfirstlane(xcd_block(blockIdx.x, gridDim.x) * P2P_WAVES + w);
    if (unit >= nleaves)
        return;
    const int lane = lane_id();
    const uint64_t lt = lanemask_lt();
    const int grp = lane >> 3, slot = lane & 7;
    const int2 pc = pieces ? pieces[unit] : make_int2(unit, 0);
    const int leaf = pc.x;
    const int v = leaf_node[leaf];
    const int64_t f = first[v];
    const int c = count[v];
    const int nbf = max(0, min(near_cnt[leaf], cap_near)) * nsub;
    const int b_lo = pieces ? pc.y * per : 0;
    const int b_hi = pieces ? min(nbf, b_lo + per) : nbf;
    const int32_t *nl = near_src + (int64_t)leaf * cap_near;
    const double *rv = recA + (int64_t)NREC * v;
    const double *Lv = Lloc + (int64_t)NLOC * v;
    int2 *R = rng[w];
    for (int sb = 0; sb < c; sb += NS) {
        double sx[NS], sy[NS], sz[NS], H4 = 0.0;
#pragma unroll
        for (int q = 0; q < NS; ++q) {
            const int64_t is = f + min(sb + q, c - 1);
            const double4 x4 = pm[is];
            sx[q] = x4.x;
            sy[q] = x4.y;
            sz[q] = x4.z;
            const double h4q = ph[is].z;
            H4 = h4q > H4 ? h4q : H4;
        }
        if (lane < NS) {
            const double4 h4 = ph[f + min(sb + lane, c - 1)];
            shh[w][lane] = make_double2(h4.x, h4.y);
        }
        // pieces of `per` source blocks: each ends with its queues drained
        // and its per-lane sums reduce-scattered, and the piece sums add up
        // in piece order (the same sums, bit for bit, whether a wavefront
        // takes all of a leaf's pieces or one piece each)
        double tot = 0.0;
        double acc[3 * NS];
        int tail[NS];  // queue fill counts; entries [tail & ~63, tail) are pending
        auto drain = [&](int q, int head, int cnt) {
            const double2 hs = shh[w][q];
            p2p_drain_f64<NS>(pm, ph, que[w][q], head, cnt, lane, nnull, sx[q], sy[q], sz[q],
                              hs.x, hs.y, acc[3 * q], acc[3 * q + 1], acc[3 * q + 2]);
        };
        for (int p0 = b_lo; p0 < b_hi; p0 += per) {
        const int nb = min(b_hi, p0 + per);
#pragma unroll
        for (int q = 0; q < 3 * NS; ++q)
            acc[q] = 0.0;
#pragma unroll
        for (int q = 0; q < NS; ++q)
            tail[q] = 0;
        for (int c0 = p0; c0 < nb; c0 += P2P_BLOCKS) {
            const int nc = min(nb - c0, P2P_BLOCKS);
            const int ne = __builtin_amdgcn_readfirstlane(
                stage_blocks_in_order(nl, c0, nc, nsub, first, count, lane, R));
            __builtin_amdgcn_wave_barrier();
            for (int kb = 0; kb < ne; kb += 8) {
                // (the latency of these loads is covered by the other
                // wavefronts of the SIMD: no registers are held for a prefetch)
                const int32_t j = (int32_t)block_src(R[kb + grp], slot, nnull);
                const double4 xj = pm[j];
                const double hj4 = ph[j].z;
                const double hmax4 = hj4 > H4 ? hj4 : H4;
#pragma unroll
                for (int q = 0; q < NS; ++q) {
                    if (SKIP && q > 0 && sb + q >= c)
                        continue;
                    const double dx = sx[q] - xj.x, dy = sy[q] - xj.y, dz = sz[q] - xj.z;
                    const double r2 = dx * dx + dy * dy + dz * dz;
                    // (every lane is active here: the softened mask is the
                    // complement of the Newtonian one)
                    const bool newt = !(r2 < hmax4);
                    const uint64_t bal = ~__ballot(newt);
                    const double fm = newt ? m_over_r3(r2, xj.w) : 0.0;
                    acc[3 * q] -= fm * dx;
                    acc[3 * q + 1] -= fm * dy;
                    acc[3 * q + 2] -= fm * dz;
                    if (bal) {
                        // possibly softened pairs leave the step for the sink's queue
                        const int t0 = tail[q];
                        if (!newt)
                            que[w][q][(t0 + __popcll(bal & lt)) & (P2P_QCAP - 1)] = j;
                        tail[q] = t0 + __popcll(bal);
                        // a queue that has gathered another 64 pairs is evaluated
                        if ((tail[q] >> 6) != (t0 >> 6)) {
                            __builtin_amdgcn_wave_barrier();
                            drain(q, t0 & ~63, 64);
                        }
                    }
                }
            }
            __builtin_amdgcn_wave_barrier();
        }
#pragma unroll
        for (int q = 0; q < NS; ++q)
            if (tail[q] & 63)
                drain(q, tail[q] & ~63, tail[q] & 63);
        __builtin_amdgcn_wave_barrier();
        tot += reduce_scatter24<double>(acc, lane);
        }
        const int idx = rs24_index(lane);
        const int q = idx / 3, comp = idx - 3 * (idx / 3);
        if (pieces && nbf > per) {
            if (idx >= 0 && (lane & 1) == 0 && sb + q < c)
                part[(int64_t)unit * part_stride + 3 * (sb + q) + comp] = tot;
        } else if (idx >= 0 && (lane & 1) == 0 && sb + q < c) {
            // component comp of eq. (8) at sink q
            double sxq = sx[0], syq = sy[0], szq = sz[0];
#pragma unroll
            for (int r = 1; r < NS; ++r)
                if (q == r) {
                    sxq = sx[r];
                    syq = sy[r];
                    szq = sz[r];
                }
            double Lr[19];
#pragma unroll
            for (int k = 0; k < 19; ++k)
                Lr[k] = Lv[k];
            double fx, fy, fz;
            l2p<double>(Lr, sxq - rv[0], syq - rv[1], szq - rv[2], fx, fy, fz);
            const double far_c = comp == 0 ? fx : (comp == 1 ? fy : fz);
            const int64_t o = 3 * (int64_t)perm[f + sb + q] + comp;
            aout[o] = G * (far_c + tot);
        }
        __builtin_amdgcn_wave_barrier();
    }
}

// ---------------------------------------------------------------- FP32 form
__device__ __forceinline__ float m4g_f32(float q, float hinv3, float u3)
{
    // both pieces are evaluated and selected (no divergent branches)
    const float p1 = hinv3 * (4.0f / 3.0f + q * q * (-1.2f + 0.5f * q));
    const float p2 = hinv3 * (8.0f / 3.0f + q * (-3.0f + q * (1.2f - q * (1.0f / 6.0f)))) -
                     u3 * (1.0f / 15.0f);
    const float g = __builtin_unpredictable(q < 2.0f) ? p2 : u3;
    return __builtin_unpredictable(q < 1.0f) ? p1 : g;
}

// FP32 near field with leaf-relative offsets: for a sink in leaf a and a
// source in leaf b, x_i - x_j = (c_a - c_b) + (y_i - y_j) with c_a - c_b formed
// in FP64 and rounded once per leaf pair, and y = x - c_leaf stored in FP32.
// Eight sinks per pass (wave-uniform), source per lane, FP32 accumulation;
// pf[p] = (y, m), pfh[p] = (1/h, 1/h^3, 4 h^2, 0), all rounded from FP64.
// A step whose pairs all lie outside both softening supports of eqs.
// (14)-(15) takes the Newtonian form; otherwise the whole step takes the M4
// form (exact on both sides of the support).  In FP32 the M4 form costs
// little more than the Newtonian one, so, unlike the FP64 kernel, no pair is
// deferred: instead the blocks of a chunk of the near list whose leaves lie
// within CLOSE_FRAC of the bound of eq. (5),
//   |c_a - c_b| < CLOSE_FRAC ((s_a + s_b) + R_kern max(h_a, h_b)),
// are staged first (each group in list order), so that the softened pairs
// gather in few steps.  The order of all additions depends on the lists
// only.  Long lists are cut into pieces of `per` blocks as in the FP64
// kernel.
// It waits for its sources 40 % of the time with four wavefronts per SIMD; the
// fifth costs a few spilled registers outside the steps and pays: 345 -> 329 us
// (binary, 2^19 particles), 9.95 -> 9.32 ms (2^24), 1.63 -> 1.48 ms (Plummer,
// 2^19).  Loading a step ahead with four took 360 us and 10.2 ms.
__device__ __forceinline__ float rsq_pos_f(float x) { return __builtin_amdgcn_rsqf(x); }

constexpr int P2P_RANGES_F32 = 256;    // blocks staged in LDS per chunk
constexpr double CLOSE_FRAC2 = 0.49;   // CLOSE_FRAC = 0.7, squared

// Position of a block in the partitioned chunk; front / back are the
// wave-uniform fill positions (front grows from 0, back shrinks from nc).
__device__ __forceinline__ int close_first_slot(bool act, bool close, int &front, int &back)
{
    const uint64_t lt = lanemask_lt();
    const uint64_t mc = __ballot(act && close), mf = __ballot(act && !close);
    const int nf = __popcll(mf);
    const int pos = close ? front + __popcll(mc & lt) : back - nf + __popcll(mf & lt);
    front += __popcll(mc);
    back -= nf;
    return pos;
}

// Staged position of step block k (close blocks, then the far ones after the
// gap left by dropped empty blocks).
__device__ __forceinline__ int skip_gap(int k, int front, int gap)
{
    return k < front ? k : k + gap;
}

template <bool SKIP>
__global__ __launch_bounds__(P2P_WG) __attribute__((amdgpu_waves_per_eu(5, 8))) void k_p2p_src_f32(
    const float4 *__restrict__ pf, const float4 *__restrict__ pfh,
    const int32_t *__restrict__ first,
    const int32_t *__restrict__ count, const int32_t *__restrict__ leaf_node, int nleaves,
    const int32_t *__restrict__ near_cnt, const int32_t *__restrict__ near_src, int cap_near,
    int nsub, const float *__restrict__ Lloc, const double *__restrict__ recA,
    const int32_t *__restrict__ perm, float G, double r_kern, float *aout,
    const int2 *__restrict__ pieces, int per, float *part, int part_stride)
{
    constexpr int NS = P2P_NS;
    constexpr int NR = P2P_RANGES_F32;
    __shared__ int2 rng[P2P_WAVES][NR + 8];
    __shared__ float4 dcs[P2P_WAVES][NR + 8];
    const int w = threadIdx.x >> 6;
    const int unit =
        __builtin_amdgcn_readfirstlane(xcd_block(blockIdx.x, gridDim.x) * P2P_WAVES + w);
    if (unit >= nleaves)
        return;
    const int lane = lane_id();
    const int grp = lane >> 3, slot = lane & 7;
    const int2 pc = pieces ? pieces[unit] : make_int2(unit, 0);
    const int leaf = pc.x;
    const int v = leaf_node[leaf];
    const int64_t f = first[v];
    const int c = count[v];
    const int nbf = max(0, min(near_cnt[leaf], cap_near)) * nsub;
    const int b_lo = pieces ? pc.y * per : 0;
    const int b_hi = pieces ? min(nbf, b_lo + per) : nbf;
    const int32_t *nl = near_src + (int64_t)leaf * cap_near;
    const double *rv = recA + (int64_t)NREC * v;
    const double ca0 = rv[0], ca1 = rv[1], ca2 = rv[2];
    const float *Lv = Lloc + (int64_t)NLOC * v;
    int2 *R = rng[w];
    float4 *D = dcs[w];
    for (int sb = 0; sb < c; sb += NS) {
        float sx[NS], sy[NS], sz[NS], shi[NS], sh3[NS], sh4[NS];
#pragma unroll
        for (int q = 0; q < NS; ++q) {
            const int64_t is = f + min(sb + q, c - 1);
            const float4 y4 = pf[is];
            const float4 h4 = pfh[is];
            sx[q] = y4.x;
            sy[q] = y4.y;
            sz[q] = y4.z;
            shi[q] = h4.x;
            sh3[q] = h4.y;
            sh4[q] = h4.z;
        }
        float tot = 0.0f;
        for (int p0 = b_lo; p0 < b_hi; p0 += per) {
        const int nb = min(b_hi, p0 + per);
        float acc[3 * NS];
#pragma unroll
        for (int q = 0; q < 3 * NS; ++q)
            acc[q] = 0.0f;
        for (int c0 = p0; c0 < nb; c0 += NR) {
            const int nc = min(nb - c0, NR);
            // stage the source blocks of this chunk: their particle range and
            // the leaf-centre difference c_a - c_b, formed in FP64 and rounded
            // to FP32; close leaves first, empty blocks dropped, eight empty
            // blocks after the last one
            int front = 0, back = nc;
            for (int k0 = 0; k0 < nc; k0 += 64) {
                const int k = k0 + lane;
                int2 r = make_int2(0, 0);
                float4 d = make_float4(0.f, 0.f, 0.f, 0.f);
                bool close = false;
                if (k < nc) {
                    const int e = (c0 + k) / nsub, u = (c0 + k) - e * nsub;
                    const int bn = nl[e];
                    r = make_int2(first[bn] + 8 * u, max(0, min(8, count[bn] - 8 * u)));
                    const double *rb = recA + (int64_t)NREC * bn;
                    const double dx = ca0 - rb[0], dy = ca1 - rb[1], dz = ca2 - rb[2];
                    d = make_float4((float)dx, (float)dy, (float)dz, 0.f);
                    const double t5 = (rv[4] + rb[4]) + r_kern * fmax(rv[5], rb[5]);
                    close = dx * dx + dy * dy + dz * dz < CLOSE_FRAC2 * t5 * t5;
                }
                const bool keep = r.y > 0;
                const int pos = close_first_slot(keep, close, front, back);
                if (keep) {
                    R[pos] = r;
                    D[pos] = d;
                }
            }
            front = __builtin_amdgcn_readfirstlane(front);
            const int gap = __builtin_amdgcn_readfirstlane(back - front), ne = nc - gap;
            if (lane < 8) {
                R[nc + lane] = make_int2(0, 0);
                D[nc + lane] = make_float4(0.f, 0.f, 0.f, 0.f);
            }
            __builtin_amdgcn_wave_barrier();
            for (int kb = 0; kb < ne; kb += 8) {
                const int kk = skip_gap(kb + grp, front, gap);
                const int2 rg = R[kk];
                const float4 dc = D[kk];
                // a missing source reads particle 0 (an empty block's start
                // may be one past the last particle) and is then replaced by
                // a far, massless one
                const bool valid = slot < rg.y;
                const int64_t j = valid ? (int64_t)rg.x + slot : 0;
                float4 yj = pf[j];
                float4 hj = pfh[j];
                if (!valid) {
                    yj = make_float4(1e30f, 1e30f, 1e30f, 0.0f);
                    hj.z = 0.0f;
                }
#pragma unroll
                for (int q = 0; q < NS; ++q) {
                    if (SKIP && q > 0 && sb + q >= c)
                        continue;
                    const float dx = dc.x + (sx[q] - yj.x), dy = dc.y + (sy[q] - yj.y),
                                dz = dc.z + (sz[q] - yj.z);
                    const float r2 = dx * dx + dy * dy + dz * dz;
                    float fm;
                    if ((__ballot(r2 < hj.z) | __ballot(r2 < sh4[q])) == 0ull) {
                        const float u = rsq_pos_f(r2);
                        fm = yj.w * (u * u * u);
                    } else {
                        const float u = r2 > 0.0f ? rsq_pos_f(r2) : 0.0f;
                        const float r = r2 * u;
                        const float u3 = u * u * u;
                        const float gi = m4g_f32(r * shi[q], sh3[q], u3);
                        const float gj = m4g_f32(r * hj.x, hj.y, u3);
                        fm = yj.w * 0.5f * (gi + gj);
                    }
                    acc[3 * q] -= fm * dx;
                    acc[3 * q + 1] -= fm * dy;
                    acc[3 * q + 2] -= fm * dz;
                }
            }
            __builtin_amdgcn_wave_barrier();
        }
        tot += reduce_scatter24<float>(acc, lane);
        }
        const int idx = rs24_index(lane);
        const int q = idx / 3, comp = idx - 3 * (idx / 3);
        if (pieces && nbf > per) {
            if (idx >= 0 && (lane & 1) == 0 && sb + q < c)
                part[(int64_t)unit * part_stride + 3 * (sb + q) + comp] = tot;
        } else if (idx >= 0 && (lane & 1) == 0 && sb + q < c) {
            float sxq = sx[0], syq = sy[0], szq = sz[0];
#pragma unroll
            for (int r = 1; r < NS; ++r)
                if (q == r) {
                    sxq = sx[r];
                    syq = sy[r];
                    szq = sz[r];
                }
            float Lr[19];
#pragma unroll
            for (int k = 0; k < 19; ++k)
                Lr[k] = Lv[k];
            float fx, fy, fz;
            l2p<float>(Lr, sxq, syq, szq, fx, fy, fz);
            const float far_c = comp == 0 ? fx : (comp == 1 ? fy : fz);
            const int64_t o = 3 * (int64_t)perm[f + sb + q] + comp;
            aout[o] = G * (far_c + tot);
        }
        __builtin_amdgcn_wave_barrier();
    }
}

// ---------------------------------------------------------------- near field, leaf <- cell lists
// The same with y cubed before the correction: (1 - e)^(-3/2) = 1 + 3/2 e +
// 15/8 e^2 + O(e^3) (y is good to about 2^-23, so the remainder is below
// 2^-66).  k15 is 1.5, in a register.
__device__ __forceinline__ double m_over_r3_k(double r2, double m, double k15)
{
    const double y = __builtin_amdgcn_rsq(r2);
    const double y2 = y * y;
    const double e = fma(-r2, y2, 1.0);
    const double my3 = (m * y) * y2;
    return fma(my3 * e, fma(e, 1.875, k15), my3);
}

// Near field.  One wavefront per sink leaf (TEAM for few).  The leaf's sinks are laid over
// the lanes two by two, each pair of sinks over the g = floor(64 / pairs)
// lanes of a group, and a step takes g source particles from LDS, one per lane
// of the group (for 8 sinks: 4 groups, 16 sources, 128 pairs a step).  So every
// lane works whatever the leaf's count, the sums of a lane are six registers
// (24 with a lane per source and all sinks in every lane), and two pairs per
// lane are independent work.
//
// Sources reach LDS 64 at a time: 8 blocks of the near list (a near leaf gives
// ceil(leaf_size / 8) blocks of at most 8 particles), a lane per particle.
// Each is tested against the bounding box of the leaf: one whose distance from
// the box is beyond the softening supports of eqs. (14)-(15) of itself and of
// every sink is Newtonian for all of them and goes to one ring buffer, the
// others go to a second one.  (The box holds its particles however it rounds,
// so a pair at r = 0 never reaches the first ring, whose steps divide by r.)  A step over the first ring is m / r^3 without a
// test; a step over the second one takes the M4 kernel, which is exact on both
// sides of the support, if any of its pairs is inside one.  A ring is emptied
// g sources at a time, the rest stays for the next 64, so missing particles
// and short blocks cost no lanes.
//
// VALU issue bounds it (89 % of its cycles, 44 instructions per 64 pairs: 12 to
// bring sources to LDS and for the leaf's start and end, 13 for the Newtonian
// steps, 17 for the second ring, which holds a third of the pairs with
// 58-neighbour smoothing lengths).  Measured against k_p2p_src_f64, whose lanes
// each take a source and all (eight, wave-uniform) sinks: 560 -> 509 us (binary,
// 2^19), 4.56 -> 4.16 ms (clumpy cube, 2^22), 497 -> 304 us where leaves hold 4
// to 10 particles (centre-of-mass tree, 200003).
//
// It takes the lists of the leaf <- cell walk.  Those of the mutual walk stay
// with k_p2p_src_f64, which keeps their forces the same to the bit: a choice, since
// the rounding that is left of their sum is bounded whatever the order.
//
// The order of all additions depends on the lists only, so results are bitwise
// reproducible.
// One wavefront per workgroup (the leaves' near lists differ in length, and a
// workgroup's slots are only freed when its last wavefront ends), or a team of
// TEAM, each with a share of the blocks and rings of its own, for few leaves.
constexpr int P2P_SINKS = 16;  // sinks per pass, at most
constexpr int P2P_RING = 128;  // sources a ring holds: less than g <= 64 left over, plus 64

// Lanes per pair of sinks for 1..8 pairs: floor(64 / pairs).
__device__ __forceinline__ int lanes_per_pair(int pairs)
{
    return (int)((0x08090a0c10152040ull >> (8 * (pairs - 1))) & 0xffull);
}

// Rotation by N lanes within each row of 16 lanes.
template <int N>
__device__ __forceinline__ double row_ror(double v)
{
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), 0x120 | N, 0xf, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), 0x120 | N, 0xf, 0xf, false);
    return __hiloint2double(hi, lo);
}
__device__ __forceinline__ double row_sum(double v)
{
    v += row_ror<8>(v);
    v += row_ror<4>(v);
    v += row_ror<2>(v);
    v += row_ror<1>(v);
    return v;
}

// The two rings of sources in LDS (x, y, z, m), and 1/h of the second one.
// An index is ring * P2P_RING + position.
struct NearRings {
    double2 xy[2 * P2P_RING], zm[2 * P2P_RING];
    double hi[P2P_RING];
};

template <int TEAM>
__global__ __launch_bounds__(64 * TEAM)
    __attribute__((amdgpu_waves_per_eu(4, 8))) void k_p2p_rings(
    const double2 *__restrict__ pxy, const double2 *__restrict__ pzm,
    const double *__restrict__ phi, const double *__restrict__ lbox, const int32_t *__restrict__ first,
    const int32_t *__restrict__ count, const int32_t *__restrict__ leaf_node, int nunits,
    const int32_t *__restrict__ near_cnt, const int32_t *__restrict__ near_src, int cap_near,
    int nsub, const double *__restrict__ Lloc, const double *__restrict__ recA,
    const int32_t *__restrict__ perm, double G, double *aout, const int2 *__restrict__ pieces,
    int per, double *part, int part_stride)
{
    constexpr int RM = P2P_RING - 1;
    __shared__ NearRings rings[TEAM];
    __shared__ double team[TEAM][64];  // sums of the team's wavefronts
    const int unit = __builtin_amdgcn_readfirstlane(xcd_block(blockIdx.x, gridDim.x));
    if (unit >= nunits)
        return;
    const int lane = lane_id();
    const int w = TEAM > 1 ? __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) : 0;
    NearRings &R = rings[w];
    const int grp = lane >> 3, slot = lane & 7;
    const int2 pc = pieces ? pieces[unit] : make_int2(unit, 0);
    const int leaf = pc.x;
    const int v = leaf_node[leaf];
    const int64_t f = first[v];
    const int c = count[v];
    const int nbf = max(0, min(near_cnt[leaf], cap_near)) * nsub;
    const int b_lo = pieces ? pc.y * per : 0;
    const int b_hi = pieces ? min(nbf, b_lo + per) : nbf;
    const int32_t *nl = near_src + (int64_t)leaf * cap_near;
    const double *rv = recA + (int64_t)NREC * v;
    const double *Lv = Lloc + (int64_t)NLOC * v;
    const double *lb = lbox + (int64_t)LBOX * leaf;
    const double bx = lb[0], by = lb[1], bz = lb[2], wx = lb[3], wy = lb[4], wz = lb[5],
                 H4 = lb[6];
    const int npass = (c + P2P_SINKS - 1) / P2P_SINKS;
    const int nsp = (c + npass - 1) / npass;  // sinks per pass
    for (int sb = 0; sb < c; sb += nsp) {
        const int cs = min(nsp, c - sb);
        const int np = (cs + 1) >> 1;      // pairs of sinks
        const int g = lanes_per_pair(np);  // lanes per pair
        const int pr = np == 4 ? lane >> 4 : min(lane / g, np - 1);
        const int k = lane - pr * g;       // k >= g: an idle lane
        double sx[2], sy[2], sz[2], shi[2];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int64_t is = f + sb + min(2 * pr + q, cs - 1);
            const double2 xy = pxy[is], zm = pzm[is];
            sx[q] = xy.x;
            sy[q] = xy.y;
            sz[q] = zm.x;
            shi[q] = phi[is];
        }
        double k15 = 1.5;
        asm("" : "+v"(k15));  // kept in a register, not set up for each pair
        // pieces of `per` source blocks: each ends with its rings emptied and
        // its sums reduced, and the piece sums add up in piece order (the
        // same sums, bit for bit, whether a wavefront takes all of a leaf's
        // pieces or one piece each)
        double tot = 0.0;
        for (int p0 = b_lo; p0 < b_hi; p0 += per) {
            const int nb = min(b_hi, p0 + per);
            double a[6];
#pragma unroll
            for (int q = 0; q < 6; ++q)
                a[q] = 0.0;
            // fill and read positions of the two rings
            int tn = 0, hn = 0, tc = 0, hc = 0;
            // a step over the first ring; lanes from lim on take no source
            auto newton = [&](int lim) {
                const double2 xy = R.xy[(hn + k) & RM], zm = R.zm[(hn + k) & RM];
                double4 s = make_double4(xy.x, xy.y, zm.x, zm.y);
                const bool none = lim < 64 && k >= lim;
                if (none)
                    s = make_double4(sx[0], sy[0], sz[0], 0.0);
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    const double dx = sx[q] - s.x, dy = sy[q] - s.y, dz = sz[q] - s.z;
                    double fm = m_over_r3_k(dx * dx + dy * dy + dz * dz, s.w, k15);
                    if (none)
                        fm = 0.0;
                    a[3 * q] -= fm * dx;
                    a[3 * q + 1] -= fm * dy;
                    a[3 * q + 2] -= fm * dz;
                }
            };
            auto soft = [&](int lim) {
                const int i = (hc + k) & RM;
                const double2 xy = R.xy[P2P_RING + i], zm = R.zm[P2P_RING + i];
                double4 s = make_double4(xy.x, xy.y, zm.x, zm.y);
                double hj = R.hi[i];
                if (lim < 64 && k >= lim) {  // u = 0 or finite: adds zero
                    s = make_double4(sx[0], sy[0], sz[0], 0.0);
                    hj = 0.0;
                }
                double dx[2], dy[2], dz[2], u[2], qi[2], qj[2];
                bool in = false;
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    dx[q] = sx[q] - s.x;
                    dy[q] = sy[q] - s.y;
                    dz[q] = sz[q] - s.z;
                    const double r2 = dx[q] * dx[q] + dy[q] * dy[q] + dz[q] * dz[q];
                    u[q] = r2 > 0.0 ? rsqrt_pos(r2) : 0.0;
                    const double r = r2 * u[q];
                    qi[q] = r * shi[q];
                    qj[q] = r * hj;
                    in = in || fmin(qi[q], qj[q]) < 2.0;
                }
                const bool any = __ballot(in && k < g) != 0ull;
                const double mh = 0.5 * s.w, hj3 = hj * hj * hj;
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    const double u3 = u[q] * u[q] * u[q];
                    double fm = s.w * u3;
                    if (any)
                        fm = mh * (m4g_f64(qi[q], shi[q] * shi[q] * shi[q], u3) +
                                   m4g_f64(qj[q], hj3, u3));
                    a[3 * q] -= fm * dx[q];
                    a[3 * q + 1] -= fm * dy[q];
                    a[3 * q + 2] -= fm * dz[q];
                }
            };
            const int wb = team_first<TEAM>(p0, nb, w), we = team_first<TEAM>(p0, nb, w + 1);
            for (int c0 = wb; c0 < we; c0 += 64) {
                // the particle ranges of 64 blocks, a lane each, the empty
                // ones moved behind the others
                int rx = 0, ry = 0;
                if (c0 + lane < we) {
                    const int e = (c0 + lane) / nsub, u = (c0 + lane) - e * nsub;
                    const int bn = nl[e];
                    rx = first[bn] + 8 * u;
                    ry = max(0, min(8, count[bn] - 8 * u));
                }
                const uint64_t mk = __ballot(ry > 0);
                const int ne = __popcll(mk);
                if (nsub > 1) {
                    const int to = 4 * (ry > 0 ? below(mk, 0) : below(~mk, ne));
                    rx = __builtin_amdgcn_ds_permute(to, rx);
                    ry = __builtin_amdgcn_ds_permute(to, ry);
                }
                struct Src {
                    int j;
                    double2 xy, zm;
                    double hi;
                };
                auto load = [&](int kb) {  // the lane's source of 8 blocks from kb on
                    const int n = __builtin_amdgcn_ds_bpermute(4 * (kb + grp), ry);
                    const int s0 = __builtin_amdgcn_ds_bpermute(4 * (kb + grp), rx);
                    Src r;
                    r.j = slot < n ? s0 + slot : -1;
                    const int64_t i = max(r.j, 0);
                    r.xy = pxy[i];
                    r.zm = pzm[i];
                    r.hi = phi[i];
                    return r;
                };
                for (int kb = 0; kb < ne; kb += 8) {
                    const Src r = load(kb);
                    const double x = r.xy.x, y = r.xy.y, z = r.zm.x;
                    const double ex = fmax(fabs(x - bx) - wx, 0.0),
                                 ey = fmax(fabs(y - by) - wy, 0.0),
                                 ez = fmax(fabs(z - bz) - wz, 0.0);
                    const double d2 = ex * ex + ey * ey + ez * ez;
                    const bool act = r.j >= 0, far = d2 >= H4 && (d2 * r.hi) * r.hi >= 4.0;
                    const uint64_t ma = __ballot(act), mf = __ballot(far);
                    const uint64_t mn = ma & mf, mc = ma & ~mf;
                    const int i = far ? below(mn, tn) & RM : (below(mc, tc) & RM) | P2P_RING;
                    if (act) {
                        R.xy[i] = r.xy;
                        R.zm[i] = r.zm;
                        if (!far)
                            R.hi[i & RM] = r.hi;
                    }
                    tn += __popcll(mn);
                    tc += __popcll(mc);
                    __builtin_amdgcn_wave_barrier();
                    for (; tn - hn >= g; hn += g)
                        newton(64);
                    for (; tc - hc >= g; hc += g)
                        soft(64);
                    __builtin_amdgcn_wave_barrier();
                }
            }
            if (tn > hn)
                newton(tn - hn);
            if (tc > hc)
                soft(tc - hc);
            __builtin_amdgcn_wave_barrier();
            // sums over the lanes of a group; lane k < 6 keeps value k
            if (g == 16) {
#pragma unroll
                for (int q = 0; q < 6; ++q)
                    a[q] = row_sum(a[q]);
            } else {
                for (int off = 32; off >= 1; off >>= 1) {
                    if (off >= g)
                        continue;
                    const bool take = k < off && k + off < g;
#pragma unroll
                    for (int q = 0; q < 6; ++q) {
                        const double o = __shfl_down(a[q], off);
                        a[q] += take ? o : 0.0;
                    }
                }
#pragma unroll
                for (int q = 0; q < 6; ++q)
                    a[q] = __shfl(a[q], pr * g);
            }
            double val = a[0];
#pragma unroll
            for (int q = 1; q < 6; ++q)
                val = k == q ? a[q] : val;
            tot += team_sum<TEAM>(val, team, w, lane);
        }
        const int q = k >= 3 ? 1 : 0, comp = k - 3 * q;
        if (w == 0 && k < 6 && 2 * pr + q < cs) {
            const int si = sb + 2 * pr + q;
            if (pieces && nbf > per) {
                part[(int64_t)unit * part_stride + 3 * si + comp] = tot;
            } else {
                // component comp of eq. (8) at the sink
                double y0 = q ? sx[1] : sx[0], y1 = q ? sy[1] : sy[0], y2 = q ? sz[1] : sz[0];
                y0 -= rv[0];
                y1 -= rv[1];
                y2 -= rv[2];
                double Lr[19];
#pragma unroll
                for (int i = 0; i < 19; ++i)
                    Lr[i] = Lv[i];
                double fx, fy, fz;
                l2p<double>(Lr, y0, y1, y2, fx, fy, fz);
                const double far_c = comp == 0 ? fx : (comp == 1 ? fy : fz);
                aout[3 * (int64_t)perm[f + si] + comp] = G * (far_c + tot);
            }
        }
    }
}

// ---------------------------------------------------------------- mutual walk
// Far field of the mutual walk: M2L into every sink cell over its CSR range
// of the sorted (sink, source) keys, then L2L down to the leaves.
template <int FORM>
__device__ __forceinline__ void m2l_node_src(const double *recA, const double *recQ,
                                             const float *, int b, double c0, double c1,
                                             double c2, double *L)
{
    const double4 cb = *(const double4 *)(recA + (int64_t)NREC * b);
    const double *qb = recQ + (int64_t)NREC * b;
    const double2 q01 = *(const double2 *)qb, q23 = *(const double2 *)(qb + 2),
                  q45 = *(const double2 *)(qb + 4);
    const double Q[6] = {q01.x, q01.y, q23.x, q23.y, q45.x, q45.y};
    m2l_acc<double, FORM>(c0 - cb.x, c1 - cb.y, c2 - cb.z, cb.w, Q, L);
}
template <int FORM>
__device__ __forceinline__ void m2l_node_src(const double *recA, const double *,
                                             const float *recF, int b, double c0, double c1,
                                             double c2, float *L)
{
    const double4 cb = *(const double4 *)(recA + (int64_t)NREC * b);
    const float4 f0 = *(const float4 *)(recF + (int64_t)NREC * b);
    const float4 f1 = *(const float4 *)(recF + (int64_t)NREC * b + 4);
    const float Q[6] = {f0.y, f0.z, f0.w, f1.x, f1.y, f1.z};
    m2l_acc<float, FORM>((float)(c0 - cb.x), (float)(c1 - cb.y), (float)(c2 - cb.z), f0.x, Q, L);
}

// 16 lanes per sink cell (all cells; zero where the range is empty).
template <typename T, int FORM>
__global__ __launch_bounds__(256) void k_m2l_node(const double *__restrict__ recA,
                                                  const double *__restrict__ recQ,
                                                  const float *__restrict__ recF, int nnodes,
                                                  const int64_t *__restrict__ fstart,
                                                  const int64_t *__restrict__ fend,
                                                  const uint64_t *__restrict__ keys,
                                                  uint64_t mask, T *Lown)
{
    const int v = (blockIdx.x * 256 + threadIdx.x) >> 4;
    const int sub = threadIdx.x & 15;
    const bool valid = v < nnodes;
    const double *rv = recA + (int64_t)NREC * (valid ? v : 0);
    const double c0 = rv[0], c1 = rv[1], c2 = rv[2];
    T L[19];
#pragma unroll
    for (int k = 0; k < 19; ++k)
        L[k] = T(0);
    const int64_t e0 = valid ? fstart[v] : 0, e1 = valid ? fend[v] : 0;
    for (int64_t k = e0 + sub; k < e1; k += 16)
        m2l_node_src<FORM>(recA, recQ, recF, (int)(keys[k] & mask), c0, c1, c2, L);
#pragma unroll
    for (int off = 8; off >= 1; off >>= 1)
#pragma unroll
        for (int k = 0; k < 19; ++k)
            L[k] += __shfl_xor(L[k], off);
    if (valid && sub == 0) {
        T *o = Lown + (int64_t)NLOC * v;
#pragma unroll
        for (int k = 0; k < 19; ++k)
            o[k] = L[k];
        o[19] = T(0);
    }
}

// One thread per listed cell: descend from the root (pre-order ids: a cell
// lies in the left subtree of v iff its id is below right[v]), at each step
// shifting the parent's total expansion to the child's centre of mass and
// adding the child's own M2L sum.  The forces need the leaves' totals (for
// L2P); the reverse pass also lists the internal cells.
template <typename T>
__global__ __launch_bounds__(256) void k_l2l_chain(const double *__restrict__ recA,
                                                   const int32_t *__restrict__ left,
                                                   const int32_t *__restrict__ right,
                                                   const int32_t *__restrict__ nodes, int count,
                                                   const T *__restrict__ Lown, T *Lout)
{
    const int g = blockIdx.x * 256 + threadIdx.x;
    if (g >= count)
        return;
    const int u = nodes[g];
    T L[19];
#pragma unroll
    for (int k = 0; k < 19; ++k)
        L[k] = Lown[k];
    double p0 = recA[0], p1 = recA[1], p2 = recA[2];
    // the next cell on the path and its centre and own sum are loaded while
    // the current shift computes
    int ch = 0;
    double q0 = 0.0, q1 = 0.0, q2 = 0.0;
    T lo[19];
    if (u != 0) {
        ch = u < right[0] ? left[0] : right[0];
        const double *rc = recA + (int64_t)NREC * ch;
        q0 = rc[0];
        q1 = rc[1];
        q2 = rc[2];
#pragma unroll
        for (int k = 0; k < 19; ++k)
            lo[k] = Lown[(int64_t)NLOC * ch + k];
    }
    while (ch != 0) {
        int nx = 0;
        double n0 = 0.0, n1 = 0.0, n2 = 0.0;
        T ln[19];
        if (ch != u) {
            nx = u < right[ch] ? left[ch] : right[ch];
            const double *rc = recA + (int64_t)NREC * nx;
            n0 = rc[0];
            n1 = rc[1];
            n2 = rc[2];
#pragma unroll
            for (int k = 0; k < 19; ++k)
                ln[k] = Lown[(int64_t)NLOC * nx + k];
        }
        l2l_shift<T>(L, (T)(q0 - p0), (T)(q1 - p1), (T)(q2 - p2));
#pragma unroll
        for (int k = 0; k < 19; ++k)
            L[k] = lo[k] + L[k];
        p0 = q0;
        p1 = q1;
        p2 = q2;
        ch = nx;
        q0 = n0;
        q1 = n1;
        q2 = n2;
#pragma unroll
        for (int k = 0; k < 19; ++k)
            lo[k] = ln[k];
    }
    T *o = Lout + (int64_t)NLOC * u;
#pragma unroll
    for (int k = 0; k < 19; ++k)
        o[k] = L[k];
    o[19] = T(0);
}

template <int FORM>
static void far_mutual(Tree &t, bool fp64, hipStream_t s)
{
    const Topology &T = t.topo;
    const MutualLists &M = t.mw;
    const uint64_t mask = (1ull << mutual_key_bits(t)) - 1ull;
    const int gm = (int)(((int64_t)T.nnodes * 16 + 255) / 256);
    const int gl = (T.nleaves + 255) / 256;
    if (fp64) {
        k_m2l_node<double, FORM><<<gm, 256, 0, s>>>(t.recA, t.recQ, t.recF, T.nnodes, M.fstart,
                                                    M.fend, M.far_sorted, mask, M.Lown);
        k_l2l_chain<double><<<gl, 256, 0, s>>>(t.recA, t.left, t.right, t.leaf_node, T.nleaves,
                                               M.Lown, t.L);
    } else {
        k_m2l_node<float, FORM><<<gm, 256, 0, s>>>(t.recA, t.recQ, t.recF, T.nnodes, M.fstart,
                                                   M.fend, M.far_sorted, mask, M.Lownf);
        k_l2l_chain<float><<<gl, 256, 0, s>>>(t.recA, t.left, t.right, t.leaf_node, T.nleaves,
                                              M.Lownf, t.Lf);
    }
}

static hipError_t far_mutual_form(Tree &t, bool fp64, hipStream_t s)
{
    if (t.p.expansion == FMM_EXPANSION_DEHNEN)
        far_mutual<FMM_EXPANSION_DEHNEN>(t, fp64, s);
    else
        far_mutual<FMM_EXPANSION_PHANTOM>(t, fp64, s);
    return hipGetLastError();
}

hipError_t launch_far_mutual(Tree &t, hipStream_t s)
{
    return far_mutual_form(t, t.p.precision == FMM_FP64, s);
}

// FP64 totals of the internal cells from the FP64 M2L sums (mutual walk).
hipError_t launch_l2l_internal(Tree &t, hipStream_t s)
{
    const Topology &T = t.topo;
    const int n_int = T.nnodes - T.nleaves;
    if (n_int > 0)
        k_l2l_chain<double><<<(n_int + 255) / 256, 256, 0, s>>>(t.recA, t.left, t.right,
                                                               t.int_nodes, n_int, t.mw.Lown, t.L);
    return hipGetLastError();
}

template <int FORM>
static void far_leaf(Tree &t, bool fp64, hipStream_t s)
{
    const int nl = t.topo.nleaves;
    const bool pc = use_pieces(t);
    const int nu = pc ? (int)t.pfar.n : nl;
    const int g = (int)(((int64_t)nu * M2L_LANES + 255) / 256);
    const int2 *pl = pc ? t.pfar.list : nullptr;
    const int per = (int)t.far_piece_entries;
    const int extra = pc ? nu - nl : 0;
    if (fp64) {
        auto run = [&](auto kernel) {
            kernel<<<g, 256, 0, s>>>(t.recA, t.recQ, t.recF, t.leaf_node, nu, t.far_cnt, t.far_src,
                                     (int)t.cap_far, t.L, pl, per, (double *)t.pfar.part);
        };
        if (FORM == FMM_EXPANSION_PHANTOM && t.p.precision != FMM_FP32)
            run(k_m2l_leaf<double, FORM, FORM == FMM_EXPANSION_PHANTOM>);
        else
            run(k_m2l_leaf<double, FORM, false>);
        if (extra > 0)
            k_m2l_fold<double><<<(extra + 255) / 256, 256, 0, s>>>(
                t.leaf_node, t.pfar.off, t.pfar.list, extra, (const double *)t.pfar.part, t.L);
    } else {
        k_m2l_leaf<float, FORM, false><<<g, 256, 0, s>>>(
            t.recA, t.recQ, t.recF, t.leaf_node, nu, t.far_cnt, t.far_src, (int)t.cap_far, t.Lf,
            pl, per, (float *)t.pfar.part);
        if (extra > 0)
            k_m2l_fold<float><<<(extra + 255) / 256, 256, 0, s>>>(
                t.leaf_node, t.pfar.off, t.pfar.list, extra, (const float *)t.pfar.part, t.Lf);
    }
}

static hipError_t far_leaves(Tree &t, bool fp64, hipStream_t s)
{
    if (t.p.expansion == FMM_EXPANSION_DEHNEN)
        far_leaf<FMM_EXPANSION_DEHNEN>(t, fp64, s);
    else
        far_leaf<FMM_EXPANSION_PHANTOM>(t, fp64, s);
    return hipGetLastError();
}

hipError_t launch_far(Tree &t, hipStream_t s)
{
    return far_leaves(t, t.p.precision == FMM_FP64, s);
}

hipError_t launch_far_f64(Tree &t, hipStream_t s)
{
    return t.lists_policy == FMM_WALK_MUTUAL ? far_mutual_form(t, true, s) : far_leaves(t, true, s);
}

// The near field of leaves whose lists were split: each leaf's piece sums
// in piece order, then L2P (eq. (8)) and the output, exactly as the kernels
// finish an unsplit leaf.  One wavefront per extra list entry; the one
// holding piece 1 of its leaf folds it, lanes over the leaf's 3 x count
// values.
template <typename T>
__global__ __launch_bounds__(256) void k_p2p_fold(
    const int32_t *__restrict__ leaf_node, const int2 *__restrict__ list, int extra,
    const int32_t *__restrict__ first, const int32_t *__restrict__ count,
    const int64_t *__restrict__ off, const T *__restrict__ part, int stride,
    const T *__restrict__ Lloc, const double *__restrict__ recA, const double4 *__restrict__ pm,
    const float4 *__restrict__ pf, const int32_t *__restrict__ perm, T G, T *aout)
{
    const int e = (blockIdx.x * 256 + threadIdx.x) >> 6;
    if (e >= extra || list[e].y != 1)
        return;
    const int lf = list[e].x;
    const int lane = lane_id();
    const int v = leaf_node[lf];
    const int64_t f = first[v];
    const int c = count[v];
    const int np = (int)(off[lf + 1] - off[lf]);
    const double *rv = recA + (int64_t)NREC * v;
    const T *Lv = Lloc + (int64_t)NLOC * v;
    for (int i3 = lane; i3 < 3 * c; i3 += 64) {
        T tot = T(0);
        for (int q = 0; q < np; ++q)
            tot += part[piece_pos(off, extra, lf, q) * stride + i3];
        const int i = i3 / 3, comp = i3 - 3 * (i3 / 3);
        T Lr[19];
#pragma unroll
        for (int k = 0; k < 19; ++k)
            Lr[k] = Lv[k];
        T fx, fy, fz;
        if constexpr (sizeof(T) == 8) {
            const double4 x4 = pm[f + i];
            l2p<double>(Lr, x4.x - rv[0], x4.y - rv[1], x4.z - rv[2], fx, fy, fz);
        } else {
            const float4 y4 = pf[f + i];
            l2p<float>(Lr, y4.x, y4.y, y4.z, fx, fy, fz);
        }
        const T far_c = comp == 0 ? fx : (comp == 1 ? fy : fz);
        aout[3 * (int64_t)perm[f + i] + comp] = G * (far_c + tot);
    }
}

hipError_t launch_near(Tree &t, void *a, hipStream_t s)
{
    const Topology &T = t.topo;
    const int nl = T.nleaves;
    const int nsub = (T.leaf_size + 7) / 8;
    const bool pc = use_pieces(t);
    const int nu = pc ? (int)t.pnear.n : nl;
    const int2 *pl = pc ? t.pnear.list : nullptr;
    const int per = (int)t.near_piece_blocks;
    const int stride = 3 * T.leaf_size;
    const int extra = pc ? nu - nl : 0;
    // every leaf full (no absent sinks to branch over)?
    const bool full = T.leaf_size == P2P_NS && T.n == (int64_t)P2P_NS * nl;
    if (t.p.precision == FMM_FP64) {
        // (lists_policy is set after the evaluation of a tree's new lists)
        if (t.p.walk == FMM_WALK_PHANTOM) {
            const int team = nl <= NEAR_TEAM_LEAVES ? NEAR_TEAM : 1;
            (team > 1 ? k_p2p_rings<NEAR_TEAM> : k_p2p_rings<1>)<<<nu, 64 * team, 0, s>>>(
                t.pxy, t.pzm, t.phi, t.lbox, t.first, t.count, t.leaf_node, nu, t.near_cnt,
                t.near_src, (int)t.cap_near, nsub, t.L, t.recA, t.perm, t.p.G, (double *)a, pl,
                per, (double *)t.pnear.part, stride);
        } else
            (full ? k_p2p_src_f64<false> : k_p2p_src_f64<true>)<<<
                (nu + P2P_WAVES - 1) / P2P_WAVES, P2P_WG, 0, s>>>(
            t.pm, t.ph, t.first, t.count, t.leaf_node, nu, t.near_cnt, t.near_src,
            (int)t.cap_near, nsub, t.L, t.recA, t.perm, t.p.G, t.p.r_kern, T.n, (double *)a, pl,
            per, (double *)t.pnear.part, stride);
        if (extra > 0)
            k_p2p_fold<double><<<(extra + 3) / 4, 256, 0, s>>>(
                t.leaf_node, t.pnear.list, extra, t.first, t.count, t.pnear.off,
                (const double *)t.pnear.part, stride, t.L, t.recA, t.pm, t.pf, t.perm, t.p.G,
                (double *)a);
    } else {
        (full ? k_p2p_src_f32<false> : k_p2p_src_f32<true>)<<<
            (nu + P2P_WAVES - 1) / P2P_WAVES, P2P_WG, 0, s>>>(
            t.pf, t.pfh, t.first, t.count, t.leaf_node, nu, t.near_cnt, t.near_src,
            (int)t.cap_near, nsub, t.Lf, t.recA, t.perm, (float)t.p.G, t.p.r_kern, (float *)a, pl,
            per, (float *)t.pnear.part, stride);
        if (extra > 0)
            k_p2p_fold<float><<<(extra + 3) / 4, 256, 0, s>>>(
                t.leaf_node, t.pnear.list, extra, t.first, t.count, t.pnear.off,
                (const float *)t.pnear.part, stride, t.Lf, t.recA, t.pm, t.pf, t.perm,
                (float)t.p.G, (float *)a);
    }
    return hipGetLastError();
}

// Pieces per leaf of the current lists and their offsets (device; the totals
// sit at off[nleaves]).
hipError_t launch_piece_counts(Tree &t, bool far, hipStream_t s)
{
    const int nl = t.topo.nleaves;
    const int nsub = (t.topo.leaf_size + 7) / 8;
    const int g = (nl + 255) / 256;
    k_piece_count<<<g, 256, 0, s>>>(t.near_cnt, (int)t.cap_near, nl, nsub, t.near_piece_blocks,
                                    t.pnear.np);
    if (far)
        k_piece_count<<<g, 256, 0, s>>>(t.far_cnt, (int)t.cap_far, nl, 1, t.far_piece_entries,
                                    t.pfar.np);
    hipError_t e = launch_count_scan(t.pnear.np, INT32_MAX, nl, t.pnear.tsum, t.pnear.off, s);
    if (e == hipSuccess && far)
        e = launch_count_scan(t.pfar.np, INT32_MAX, nl, t.pfar.tsum, t.pfar.off, s);
    return e;
}

hipError_t launch_piece_fill(Tree &t, bool far, hipStream_t s)
{
    const int nl = t.topo.nleaves;
    const int g = (nl + 255) / 256;
    k_piece_fill<<<g, 256, 0, s>>>(t.pnear.off, t.pnear.np, nl, t.pnear.list);
    if (far)
        k_piece_fill<<<g, 256, 0, s>>>(t.pfar.off, t.pfar.np, nl, t.pfar.list);
    return hipGetLastError();
}

hipError_t launch_piece_table(const int64_t *off, const int32_t *np, int nleaves, int2 *list,
                              hipStream_t s)
{
    if (nleaves > 0)
        k_piece_fill<<<(nleaves + 255) / 256, 256, 0, s>>>(off, np, nleaves, list);
    return hipGetLastError();
}

}  // namespace fmm
