// gfx950 kernels of the adaptive-tree variant (fmm2d_adaptive.h): the evaluation
// stages of Fig. fmmStages over the four lists of the adaptive FMM.
//
// Expansions are radius-scaled as in the uniform kernels (multipole a_m / w^m, local
// b_l w^(l+1), w the cell's width), so the translations between a cell and its parent
// and the M2L between cells of one level do not depend on the level.  Every expansion
// is FP64; the near field runs in the records' precision (FP32 for the mixed form).
// Complex charge c_j = -i Gamma_j / (2 pi); conjugate velocity W = u - i v.
#include "adaptive_internal.h"
#include "device_common.h"
#include "translate.h"

#include <cmath>

namespace fmm {
namespace {

__device__ __forceinline__ double2 cell_centre(double x0, double y0, double side, int4 c)
{
    const double w = ldexp(side, -c.x);
    return make_double2(x0 + (c.y + 0.5) * w, y0 + (c.z + 0.5) * w);
}

__device__ __forceinline__ double2 cinv(double2 a)
{
    const double r = 1.0 / (a.x * a.x + a.y * a.y);
    return make_double2(a.x * r, -a.y * r);
}

// Records {alpha (z - c_leaf), Gamma, 0} for the near field and the circulations in
// sorted order for the expansions.
// The circulation of sorted particle i from its staging slot gpos2[i] (the circulations
// staged by bucket beforehand): in the near field's precision for its records, in FP64
// for the expansions.
template <typename T>
__global__ __launch_bounds__(256) void at_pack_kernel(int n, int nxcd, const int *__restrict__ gpos2,
                                                       const double *__restrict__ gamma_st, T *__restrict__ gam,
                                                       double *__restrict__ gamma_sorted)
{
    const int i = xcd_block(nxcd) * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const double g = gamma_st[gpos2[i]];
    gam[i] = (T)g;
    gamma_sorted[i] = g;
}

// The offsets z - c_leaf of the sorted particles from their leaves' centres, in the near
// field's precision (made once per tree and precision): the near field's records are
// these offsets scaled by alpha on load (SoaRec) and the circulations.
template <typename T>
__global__ __launch_bounds__(256) void at_coords_kernel(int n, const int *__restrict__ leaf_of,
                                                         const int4 *__restrict__ cell, const double2 *__restrict__ xy,
                                                         double x0, double y0, double side, c2<T> *__restrict__ pos)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const double2 c = cell_centre(x0, y0, side, cell[leaf_of[i]]);
    const double2 z = xy[i];
    pos[i] = mk<T>((T)(z.x - c.x), (T)(z.y - c.y));
}

// Charge of sorted particle j: c_j = -i Gamma_j / (2 pi), or with q the complex charge q_j of
// the adjoint pass.
__device__ __forceinline__ double2 charge(const double *__restrict__ gamma, const double2 *__restrict__ q, int j)
{
    return q ? q[j] : make_double2(0.0, -gamma[j] * kInv2Pi);
}

// P2M (stage 4) at the leaves of level >= 2, G lanes per leaf (64/G leaves per
// wavefront):
//   a_m / w^m = sum_j c_j xi_j^m,  xi_j = (z_j - c)/w,
// the G lanes over the leaf's particles, then the sums over the G lanes by halving.
template <int PMAX, int G>
__global__ __launch_bounds__(64) void at_p2m_kernel(const int *__restrict__ cells, int ncells,
                                                     const int4 *__restrict__ cell, const int2 *__restrict__ range,
                                                     const double2 *__restrict__ xy, const double *__restrict__ gamma,
                                                     const double2 *q, double x0, double y0, double side, int p,
                                                     double2 *mp, const double2 *q2, double2 *mp2)
{
    if (blockIdx.y) {  // the second set of charges
        q = q2;
        mp = mp2;
    }
    const int lane = threadIdx.x, g = lane % G;
    const int idx = blockIdx.x * (64 / G) + lane / G;
    const bool valid = idx < ncells;  // a group past the end idles (its shuffles stay inside it)
    const int k = valid ? cells[idx] : 0;
    const int4 c = cell[k];
    const int2 r = valid ? range[k] : make_int2(0, 0);
    const double w = ldexp(side, -c.x);
    const double rw = 1.0 / w;
    const double2 ctr = cell_centre(x0, y0, side, c);
    // PMAX coefficients throughout (those at m >= p are never stored): no branches on p
    constexpr int NC = 2 * PMAX;
    double acc[NC];
#pragma unroll
    for (int m = 0; m < NC; ++m) acc[m] = 0.0;
    for (int j = r.x + g; j < r.x + r.y; j += G) {
        const double2 z = xy[j];
        const double2 xi = make_double2((z.x - ctr.x) * rw, (z.y - ctr.y) * rw);
        double2 pw = charge(gamma, q, j);
#pragma unroll
        for (int m = 0; m < PMAX; ++m) {
            acc[2 * m] += pw.x;
            acc[2 * m + 1] += pw.y;
            pw = cmul<double>(pw, xi);
        }
    }
    lane_halve<double, NC, NC, G / 2>(acc, lane);
    if (valid) store_halved<double, NC, G>(acc, g, 2 * p, (double *)(mp + (int64_t)k * p));
}

// P2L from X, written to the locals of the cells with a non-empty X list before the M2L
// adds to them, G lanes per cell (64/G cells per wavefront):
//   b_l = -sum_{j in A} c_j u_j^(l+1),  u_j = w/(z_j - c),
// the G lanes over the particles of a source leaf, then the sums over the G lanes by halving.  (One thread per cell was a serial chain over the list's particles.)
template <int PMAX, int G>
__global__ __launch_bounds__(64) void at_p2l_kernel(int first, int ncells, const int4 *__restrict__ cell,
                                                     const int *__restrict__ x_off, const int *__restrict__ x_idx,
                                                     const int2 *__restrict__ range, const double2 *__restrict__ xy,
                                                     const double *__restrict__ gamma, const double2 *q, double x0,
                                                     double y0, double side, int p, double2 *lo, const double2 *q2,
                                                     double2 *lo2)
{
    if (blockIdx.y) {  // the second set of charges
        q = q2;
        lo = lo2;
    }
    const int lane = threadIdx.x, g = lane % G;
    const int t = blockIdx.x * (64 / G) + lane / G;
    const int k = first + min(t, ncells - 1);
    const int e0 = x_off[k], e1 = t < ncells ? x_off[k + 1] : e0;
    if (!__any(e0 < e1)) return;  // a group without a list idles (its shuffles stay inside it)
    const int4 c = cell[k];
    constexpr int NC = 2 * PMAX;
    double b[NC];
#pragma unroll
    for (int l = 0; l < NC; ++l) b[l] = 0.0;
    const double rw = 1.0 / ldexp(side, -c.x);
    const double2 ctr = cell_centre(x0, y0, side, c);
    for (int e = e0; e < e1; ++e) {
        const int2 r = range[x_idx[e]];
        for (int j = r.x + g; j < r.x + r.y; j += G) {
            const double2 z = xy[j];
            const double2 u = cinv(make_double2((z.x - ctr.x) * rw, (z.y - ctr.y) * rw));
            const double2 cj = charge(gamma, q, j);
            double2 ul = cmul<double>(cj, u);  // c_j u^(l+1)
#pragma unroll
            for (int l = 0; l < PMAX; ++l) {
                b[2 * l] -= ul.x;
                b[2 * l + 1] -= ul.y;
                ul = cmul<double>(ul, u);
            }
        }
    }
    lane_halve<double, NC, NC, G / 2>(b, lane);
    if (e0 < e1) store_halved<double, NC, G>(b, g, 2 * p, (double *)(lo + (int64_t)k * p));
}

// Near field (stage 9) over U.  One wavefront per work entry:
//  - a mutual item (two adjacent dense leaves of one level, or a dense leaf with itself)
//    evaluates each unordered pair once for both particles (the kernel is odd), as for
//    the uniform tree, with that level's leaf width; sums go to the per-direction slots;
//  - a target-centric unit {leaf A, first, count <= 64, log2 TP | 16 if dense} takes
//    every source leaf S of U(A) (but the same-level dense ones when flagged), the leaves
//    concatenated and staged 64 sources at a time, each moved into A's frame
//    (alpha (z_j - c_A) = record_j + alpha (c_S - c_A)).  A source leaf whose bounding box
//    is at least the cut from the unit's box skips the exponential (1 - e rounds to 1).
template <typename T>
__device__ __forceinline__ void at_target_unit(const int4 u, rec_t<T> *tile, const int4 *__restrict__ cell,
                                               const int2 *__restrict__ range, const int *__restrict__ u_off,
                                               const int *__restrict__ u_idx, const int *__restrict__ tile_start,
                                               const double4 *__restrict__ tile_box,
                                               const SoaRec<T> &rec, double x0, double y0, double side,
                                               double alpha, double cut, double scale, int dense,
                                               double2 *__restrict__ near)
{
    const int lane = threadIdx.x;
    const bool skip_dense = (u.w >> 4) != 0;
    const UnitLanes ul(lane, u.z, u.w & 15);
    const int i = u.y + min(ul.t, u.z - 1);
    const rec_t<T> ri = rec(i);
    const int A = u.x;
    const int4 cla = cell[A];
    const double2 ca = cell_centre(x0, y0, side, cla);
    const double4 tb = tile_box[tile_start[A] + ((u.y - range[A].x) >> 6)];
    const double a2 = alpha * alpha;
    double au = 0.0, av = 0.0;
    const int eend = u_off[A + 1];
    for (int e0 = u_off[A]; e0 < eend; e0 += 64) {
        // lane k: the k-th source leaf of this group of U(A)
        int s0 = 0, len = 0;
        bool far = false;
        T ox = 0, oy = 0;
        if (e0 + lane < eend) {
            const int S = u_idx[e0 + lane];
            const int4 cls = cell[S];
            const int2 r = range[S];
            s0 = r.x;
            len = skip_dense && cls.x == cla.x && r.y >= dense ? 0 : r.y;  // else in a mutual item
            const double2 cs = cell_centre(x0, y0, side, cls);
            ox = (T)(alpha * (cs.x - ca.x));  // moved into the frame of A
            oy = (T)(alpha * (cs.y - ca.y));
            if (len > 0 && len <= 64) {  // one tile (a larger leaf takes the general form)
                const double4 sb = tile_box[tile_start[S]];
                const double gx = fmax(0.0, fmax(sb.x - tb.z, tb.x - sb.z));
                const double gy = fmax(0.0, fmax(sb.y - tb.w, tb.y - sb.w));
                far = (gx * gx + gy * gy) * a2 >= cut;
            }
        }
        auto stage = [&](int e, int j) {
            const int from = __shfl(s0, e);
            const T sx = __shfl(ox, e), sy = __shfl(oy, e);
            rec_t<T> r;
            r.x = r.y = r.z = r.w = (T)0;
            if (j >= 0) {
                r = rec(from + j);
                r.x += sx;
                r.y += sy;
            }
            tile[lane] = r;
            r.z = (T)0;
            tile[64 + lane] = r;
        };
        source_batches<64>(far ? 0 : len, stage, [&](int count) {
            T fu = 0, fv = 0;
            p2p_batch<T, false>(tile, count, ul.k, ul.K, ri.x, ri.y, fu, fv);
            au += (double)fu;
            av += (double)fv;
        });
        if (__any(far))
            source_batches<64>(far ? len : 0, stage, [&](int count) {
                T fu = 0, fv = 0;
                p2p_batch<T, true>(tile, count, ul.k, ul.K, ri.x, ri.y, fu, fv);
                au += (double)fu;
                av += (double)fv;
            });
    }
    au = ul.reduce(au);
    av = ul.reduce(av);
    if (lane < u.z) near[i] = make_double2(-scale * au, scale * av);
}

template <typename T>
__global__ __launch_bounds__(64, sizeof(T) == 4 ? 8 : 4) void at_near_kernel(
    const int4 *__restrict__ work, const int4 *__restrict__ cell, const int2 *__restrict__ range,
    const int *__restrict__ u_off, const int *__restrict__ u_idx, const int *__restrict__ tile_start,
    const double4 *__restrict__ tile_box, const int *__restrict__ leaf_start, const int *__restrict__ leaf_tile,
    const float4 *__restrict__ tile_box_leaf, const c2<T> *__restrict__ pos, const T *__restrict__ gam, double x0,
    double y0, double side, double alpha, double cut, double scale, int dense, int64_t n,
    double2 *__restrict__ near, c2<T> *__restrict__ slots)
{
    __shared__ NearLds<T, kVelocity> lds;
    const SoaRec<T> rec{pos, gam, (T)alpha};  // records alpha (z - c_leaf), Gamma
    const int4 u = work[blockIdx.x];
    if (u.w & kMutualItem) {
        const double step = alpha * ldexp(side, -(u.w >> 9));
        mutual_item<kVelocity>(u, lds, rec,
                               MutualTree{leaf_start, leaf_tile, tile_box_leaf, (float)(cut / (step * step)), 0.0f},
                               MutualParts{}, (T)step, n, slots, (T *)nullptr);
    } else {
        at_target_unit<T>(u, lds.a, cell, range, u_off, u_idx, tile_start, tile_box, rec, x0, y0, side, alpha, cut,
                          scale, dense, near);
    }
}

// Stages 8 + 10: L2P from the leaf's local expansion (level >= 2),
//   W += (1/w) sum_l b_l xi^l;  M2P from W(leaf),  W += (1/w_D) sum_m a_m zeta^-(m+1);
// (u, v) = near + (Re W, -Im W), scattered to user order.
template <typename TS>
__global__ __launch_bounds__(256) void at_finalize_kernel(int n, const int *__restrict__ perm,
                                                           const int *__restrict__ leaf_of,
                                                           const int4 *__restrict__ cell,
                                                           const double2 *__restrict__ xy,
                                                           const int *__restrict__ w_off,
                                                           const int *__restrict__ w_idx,
                                                           const double2 *__restrict__ mp,
                                                           const double2 *__restrict__ lo, int p, double x0,
                                                           double y0, double side, const double2 *__restrict__ near,
                                                           const uint16_t *__restrict__ mask,
                                                           const c2<TS> *__restrict__ slots, double scale,
                                                           double *__restrict__ uv, double *__restrict__ uv_near,
                                                           double *__restrict__ uv_far, double2 *__restrict__ staged,
                                                           const int *__restrict__ gpos2, int nxcd,
                                                           const double *base, double h)
{
    const int i = xcd_block(nxcd) * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int64_t o = staged ? (gpos2 ? gpos2[i] : i) : perm[i];  // issued with the first loads
    const int A = leaf_of[i];
    // near field: the target-centric part (mask bit 9) plus the slots of the mutual
    // items (bits d), in order d = 0..8 (first, so that its loads overlap the far part's)
    const double2 nr = near_from_slots<TS>(i, n, mask[A], near, slots, scale);
    const int4 c = cell[A];
    const double2 z = xy[i];
    double2 W = make_double2(0.0, 0.0);
    const int e1 = w_off[A + 1];
    int e = w_off[A], D = 0;
    int4 cd = make_int4(0, 0, 0, 0);
    if (e < e1) {
        D = w_idx[e];
        cd = cell[D];
    }
    if (c.x >= 2) {
        const double w = ldexp(side, -c.x);
        const double2 ctr = cell_centre(x0, y0, side, c);
        const double2 xi = make_double2((z.x - ctr.x) / w, (z.y - ctr.y) / w);
        const double2 acc = horner_prefetch<double>(lo + (int64_t)A * p, p, xi);
        W = make_double2(acc.x / w, acc.y / w);
    }
    for (; e < e1; ++e) {
        const double rw = 1.0 / ldexp(side, -cd.x);
        const double2 ctr = cell_centre(x0, y0, side, cd);
        const double2 *const m = mp + (int64_t)D * p;
        if (e + 1 < e1) {  // the next entry ahead of this one's products
            D = w_idx[e + 1];
            cd = cell[D];
        }
        const double2 inv = cinv(make_double2((z.x - ctr.x) * rw, (z.y - ctr.y) * rw));
        W = cmac<double>(W, horner_prefetch<double>(m, p, inv), make_double2(inv.x * rw, inv.y * rw));
    }
    if (staged) {  // at its staging slot (windows) or in sorted order
        staged[o] = make_double2(nr.x + W.x, nr.y - W.y);
        return;
    }
    if (uv) store_velocity(uv, o, make_double2(nr.x + W.x, nr.y - W.y), base, h);
    if (uv_near) {
        uv_near[2 * o] = nr.x;
        uv_near[2 * o + 1] = nr.y;
    }
    if (uv_far) {
        uv_far[2 * o] = W.x;
        uv_far[2 * o + 1] = -W.y;
    }
}

// ---------------------------------------------------------------------------------
// Adjoint (fmm_atree_velocity_backward).  q_i = dL/du_i + i dL/dv_i.  The adaptive
// operator is antisymmetric (odd near kernel over symmetric U lists, M2L over symmetric V
// lists, M2P over W the transpose of P2L over X at equal truncation), so, as for the
// uniform tree, dL/dGamma = -Im(Phi)/(2 pi) with Phi the same evaluation with charges q,
// the evaluation-position derivative comes from the near sums A, B and the derivative W'
// of the far field of the charges c, and the source-position derivative from the near
// sums with the charges q and the derivative Phi' of the far field of the charges q.
// ---------------------------------------------------------------------------------

// Adjoint charges in sorted order, FP64 and in the records' precision.
template <typename T>
__global__ __launch_bounds__(256) void at_pack_adjoint_kernel(int n, int nxcd, const int *__restrict__ gpos2,
                                                               const double2 *__restrict__ dl_st, double scale,
                                                               double2 *__restrict__ adj, c2<T> *__restrict__ qt)
{
    const int i = xcd_block(nxcd) * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const double2 d = dl_st[gpos2[i]];  // the cotangent staged by bucket
    const double2 q = make_double2(scale * d.x, scale * d.y);
    adj[i] = q;
    qt[i] = mk<T>((T)q.x, (T)q.y);
}

// Adjoint near field of one unit {leaf A, first, count <= 64, log2 TP}: every source leaf
// of U(A) in 64-particle tiles (records and adjoint charges staged in LDS), the target
// moved into the source leaf's frame, the exponential skipped on far tiles; the sums of
// the uniform tree's adjoint pair kernel, FP64 per source leaf.
template <typename T, bool SRC>
__device__ __forceinline__ void at_backward_unit(const int4 u, rec_t<T> *tile, c2<T> *qtile,
                                                 const int4 *__restrict__ cell, const int2 *__restrict__ range,
                                                 const int *__restrict__ u_off, const int *__restrict__ u_idx,
                                                 const int *__restrict__ tile_start,
                                                 const double4 *__restrict__ tile_box,
                                                 const SoaRec<T> &rec, const c2<T> *__restrict__ qt,
                                                 double x0, double y0, double side, double alpha, double cut,
                                                 T lambda, double4 *__restrict__ out_pa,
                                                 double4 *__restrict__ out_src)
{
    constexpr int NA = SRC ? 8 : 4;
    const int lane = threadIdx.x;
    const int logtp = u.w & 15;
    const int A = u.x;
    const int4 cla = cell[A];
    const double2 ca = cell_centre(x0, y0, side, cla);
    const double4 tb = tile_box[tile_start[A] + ((u.y - range[A].x) >> 6)];
    const double a2 = alpha * alpha;
    const int ebegin = u_off[A], eend = u_off[A + 1];
    int longest = 0;
    for (int e = ebegin + lane; e < eend; e += 64) longest = max(longest, range[u_idx[e]].y);
    // FP64, every source leaf one tile: staged together, in A's frame (FP32: see run_backward)
    if (sizeof(T) == 8 && !__any(longest > 64)) {
        const UnitLanes ul(lane, u.z, logtp);
        const int i = u.y + min(ul.t, u.z - 1);
        const rec_t<T> ri = rec(i);
        double sum[NA] = {};
        auto fold = [&](const T(&acc)[NA]) {
#pragma unroll
            for (int c = 0; c < NA; ++c) sum[c] += (double)acc[c];
        };
        for (int e0 = ebegin; e0 < eend; e0 += 64) {
            int s0 = 0, len = 0;
            bool far = false;
            T ox = 0, oy = 0;
            if (e0 + lane < eend) {
                const int S = u_idx[e0 + lane];
                const int2 r = range[S];
                s0 = r.x;
                len = r.y;
                const double2 cs = cell_centre(x0, y0, side, cell[S]);
                ox = (T)(alpha * (cs.x - ca.x));
                oy = (T)(alpha * (cs.y - ca.y));
                const double4 sb = tile_box[tile_start[S]];
                const double gx = fmax(0.0, fmax(sb.x - tb.z, tb.x - sb.z));
                const double gy = fmax(0.0, fmax(sb.y - tb.w, tb.y - sb.w));
                far = (gx * gx + gy * gy) * a2 >= cut;
            }
            auto stage = [&](int e, int j) {
                const int from = __shfl(s0, e);
                const T sx = __shfl(ox, e), sy = __shfl(oy, e);
                rec_t<T> r;
                r.x = r.y = r.z = r.w = (T)0;
                c2<T> q = mk<T>(0, 0);
                if (j >= 0) {
                    r = rec(from + j);
                    r.x += sx;
                    r.y += sy;
                    q = qt[from + j];
                }
                tile[lane] = r;
                qtile[lane] = q;
                r.z = (T)0;
                tile[64 + lane] = r;
                qtile[64 + lane] = mk<T>(0, 0);
            };
            source_batches<64>(far ? 0 : len, stage, [&](int count) {
                T acc[NA] = {};
                p2p_bwd_batch<T, false, SRC>(tile, qtile, count, ul.k, ul.K, ri.x, ri.y, lambda, acc);
                fold(acc);
            });
            if (__any(far))
                source_batches<64>(far ? len : 0, stage, [&](int count) {
                    T acc[NA] = {};
                    p2p_bwd_batch<T, true, SRC>(tile, qtile, count, ul.k, ul.K, ri.x, ri.y, lambda, acc);
                    fold(acc);
                });
        }
#pragma unroll
        for (int c = 0; c < NA; ++c) sum[c] = ul.reduce(sum[c]);
        if (lane < u.z) {
            out_pa[i] = make_double4(sum[0], sum[1], sum[2], sum[3]);
            if constexpr (SRC) out_src[i] = make_double4(sum[4], sum[5], sum[6], sum[7]);
        }
        return;
    }
    const int tp = 1 << logtp;
    const int t = lane & (tp - 1);
    const int k = lane >> logtp;
    const int i = u.y + min(t, u.z - 1);
    const rec_t<T> ri = rec(i);
    double sum[NA] = {};
    for (int e = u_off[A]; e < u_off[A + 1]; ++e) {
        const int S = u_idx[e];
        const int2 r = range[S];
        const double2 cs = cell_centre(x0, y0, side, cell[S]);
        const T tx = ri.x + (T)(alpha * (ca.x - cs.x));
        const T ty = ri.y + (T)(alpha * (ca.y - cs.y));
        T acc[NA] = {};
        int tt = tile_start[S];
        for (int base = r.x; base < r.x + r.y; base += 64, ++tt) {
            const int len = min(64, r.x + r.y - base);
            __syncthreads();
            if (lane < len) {
                tile[lane] = rec(base + lane);
                qtile[lane] = qt[base + lane];
            }
            const double4 sb = tile_box[tt];
            const double gx = fmax(0.0, fmax(sb.x - tb.z, tb.x - sb.z));
            const double gy = fmax(0.0, fmax(sb.y - tb.w, tb.y - sb.w));
            // beyond the exponential's cut: point-vortex terms; beyond twice the series cut: no
            // per-pair series test
            const double g2 = (gx * gx + gy * gy) * a2;
            const int cls = g2 >= cut ? 2 : g2 >= 2.0 * (double)series_cut<T>() / (double)lambda ? 1 : 0;
            __syncthreads();
            switch (logtp) {
            case 6: p2p_bwd_tile_any<T, 1, SRC>(tile, qtile, len, k, tx, ty, lambda, acc, cls); break;
            case 5: p2p_bwd_tile_any<T, 2, SRC>(tile, qtile, len, k, tx, ty, lambda, acc, cls); break;
            case 4: p2p_bwd_tile_any<T, 4, SRC>(tile, qtile, len, k, tx, ty, lambda, acc, cls); break;
            case 3: p2p_bwd_tile_any<T, 8, SRC>(tile, qtile, len, k, tx, ty, lambda, acc, cls); break;
            case 2: p2p_bwd_tile_any<T, 16, SRC>(tile, qtile, len, k, tx, ty, lambda, acc, cls); break;
            case 1: p2p_bwd_tile_any<T, 32, SRC>(tile, qtile, len, k, tx, ty, lambda, acc, cls); break;
            default: p2p_bwd_tile_any<T, 64, SRC>(tile, qtile, len, k, tx, ty, lambda, acc, cls); break;
            }
        }
#pragma unroll
        for (int c = 0; c < NA; ++c) sum[c] += (double)acc[c];
    }
    for (int o = tp; o < 64; o <<= 1)
#pragma unroll
        for (int c = 0; c < NA; ++c) sum[c] += __shfl_xor(sum[c], o);
    if (k == 0 && t < u.z) {
        out_pa[i] = make_double4(sum[0], sum[1], sum[2], sum[3]);
        if constexpr (SRC) out_src[i] = make_double4(sum[4], sum[5], sum[6], sum[7]);
    }
}

// FP32: 6 wavefronts per SIMD (5 with the source sums), as the uniform tree's adjoint.
template <typename T, bool SRC>
__global__ __launch_bounds__(64, sizeof(T) == 4 ? (SRC ? 5 : 6) : 2) void at_backward_kernel(
    const int4 *__restrict__ units, const int4 *__restrict__ cell, const int2 *__restrict__ range,
    const int *__restrict__ u_off, const int *__restrict__ u_idx, const int *__restrict__ tile_start,
    const double4 *__restrict__ tile_box, const c2<T> *__restrict__ pos, const T *__restrict__ gam,
    const c2<T> *__restrict__ qt, double x0, double y0, double side, double alpha, double cut, T lambda,
    double4 *__restrict__ out_pa, double4 *__restrict__ out_src)
{
    __shared__ rec_t<T> tile[128];
    __shared__ c2<T> qtile[128];
    const SoaRec<T> rec{pos, gam, (T)alpha};
    at_backward_unit<T, SRC>(units[blockIdx.x], tile, qtile, cell, range, u_off, u_idx, tile_start, tile_box, rec, qt,
                             x0, y0, side, alpha, cut, lambda, out_pa, out_src);
}

// The adjoint's near field over the pair force (dl_dxy without its two parts), over the
// forward's work list: its units, and its mutual items with each pair evaluated once.  FP64 alone
// (see run_backward).
template <int KIND>
__global__ __launch_bounds__(64, 3) void at_force_kernel(
    const int4 *__restrict__ work, const int4 *__restrict__ cell, const int2 *__restrict__ range,
    const int *__restrict__ u_off, const int *__restrict__ u_idx, const int *__restrict__ tile_start,
    const double4 *__restrict__ tile_box, const int *__restrict__ leaf_start, const int *__restrict__ leaf_tile,
    const float4 *__restrict__ tile_box_leaf, const SoaRec<double> rec, double x0, double y0, double side, double alpha,
    double cut, int dense, int64_t n, double2 *__restrict__ near, double *__restrict__ near_phi,
    double2 *__restrict__ slots, double *__restrict__ phi_slots)
{
    constexpr int NS = kSums<KIND>;
    __shared__ NearLds<double, KIND> lds;
    const int4 u = work[blockIdx.x];
    if (u.w & kMutualItem) {
        const double step = alpha * ldexp(side, -(u.w >> 9));
        mutual_item<KIND>(u, lds, rec,
                          MutualTree{leaf_start, leaf_tile, tile_box_leaf, (float)(cut / (step * step)), 0.0f},
                          MutualParts{}, step, n, slots, phi_slots);
        return;
    }
    const int lane = threadIdx.x;
    const bool skip_dense = (u.w >> 4) != 0;
    const UnitLanes ul(lane, u.z, u.w & 15);
    const int i = u.y + min(ul.t, u.z - 1);
    double tiqy;
    const double4 ti = load_rec<KIND>(rec, i, tiqy);
    const int A = u.x;
    const int4 cla = cell[A];
    const double2 ca = cell_centre(x0, y0, side, cla);
    const double4 tb = tile_box[tile_start[A] + ((u.y - range[A].x) >> 6)];
    double sum[NS] = {};
    const int eend = u_off[A + 1];
    for (int e0 = u_off[A]; e0 < eend; e0 += 64) {
        // lane k: the k-th source leaf of this group of U(A)
        int s0 = 0, len = 0;
        bool far = false;
        double ox = 0, oy = 0;
        if (e0 + lane < eend) {
            const int S = u_idx[e0 + lane];
            const int4 cls = cell[S];
            const int2 r = range[S];
            s0 = r.x;
            len = skip_dense && cls.x == cla.x && r.y >= dense ? 0 : r.y;  // else in a mutual item
            const double2 cs = cell_centre(x0, y0, side, cls);
            ox = alpha * (cs.x - ca.x);  // moved into the frame of A
            oy = alpha * (cs.y - ca.y);
            if (len > 0 && len <= 64) {  // one tile (a larger leaf takes the general form)
                const double4 sb = tile_box[tile_start[S]];
                const double gx = fmax(0.0, fmax(sb.x - tb.z, tb.x - sb.z));
                const double gy = fmax(0.0, fmax(sb.y - tb.w, tb.y - sb.w));
                far = (gx * gx + gy * gy) * (alpha * alpha) >= cut;
            }
        }
        auto stage = [&](int e, int j) {
            const int from = __shfl(s0, e);
            const double sx = __shfl(ox, e), sy = __shfl(oy, e);
            stage_source<KIND>(lds.a, lds.qa, rec, j >= 0 ? from + j : -1, sx, sy);
        };
        source_batches<64>(far ? 0 : len, stage, [&](int count) {
            double f[NS] = {};
            force_batch<double, KIND, 0>(lds.a, lds.qa, count, ul.k, ul.K, ti, tiqy, f);
            for (int m = 0; m < NS; ++m) sum[m] += f[m];
        });
        if (__any(far))
            source_batches<64>(far ? len : 0, stage, [&](int count) {
                double f[NS] = {};
                force_batch<double, KIND, 2>(lds.a, lds.qa, count, ul.k, ul.K, ti, tiqy, f);
                for (int m = 0; m < NS; ++m) sum[m] += f[m];
            });
    }
    for (int m = 0; m < NS; ++m) sum[m] = ul.reduce(sum[m]);
    if (lane < u.z) {
        const double ka = alpha * alpha * kInv2Pi;
        near[i] = make_double2(-ka * sum[0], ka * sum[1]);
        if constexpr (KIND == kForcePhi) near_phi[i] = sum[2];
    }
}

// Values and derivatives of two polynomials of p terms at x, by Horner's rule for both at once
// (P' x + P, then P x + a_l), the coefficients eight at a time ahead of their use.
__device__ __forceinline__ void horner_pair(const double2 *__restrict__ a, const double2 *__restrict__ b, int p,
                                            double2 x, double2 &va, double2 &da, double2 &vb, double2 &db)
{
    va = a[p - 1];
    vb = b[p - 1];
    da = db = make_double2(0.0, 0.0);
    for (int l0 = p - 2; l0 >= 0; l0 -= 8) {
        double2 ca[8], cb[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int l = max(l0 - k, 0);
            ca[k] = a[l];
            cb[k] = b[l];
        }
#pragma unroll
        for (int k = 0; k < 8; ++k)
            if (l0 - k >= 0) {
                da = cmac<double>(va, da, x);
                va = cmac<double>(ca[k], va, x);
                db = cmac<double>(vb, db, x);
                vb = cmac<double>(cb[k], vb, x);
            }
    }
}

// Far field of the adjoint at z in leaf A (FP64): the derivative dw of the charges c's field, the
// value phi and the derivative dphi of the charges q's, from the scaled expansions
//   L2P  (1/w) P(xi),  derivative (1/w^2) P'(xi),   P(x) = sum_l b_l x^l,  xi = (z - c_A)/w;
//   M2P  (1/w_D) x P(x),  derivative -(x/w_D)^2 (P + x P')(x),   x = w_D/(z - c_D),
// over D in W(A).  Both fields in one walk of the list, the next cell of it loaded ahead: bound
// by the chain list, cell, coefficients, Horner, which three walks had three times (150001
// clustered particles: 100 us, 60 in one walk).
__device__ __forceinline__ void far_adjoint(int A, int4 c, double2 z, const int *__restrict__ w_off,
                                            const int *__restrict__ w_idx, const int4 *__restrict__ cell,
                                            const double2 *__restrict__ mp, const double2 *__restrict__ lo,
                                            const double2 *__restrict__ mp2, const double2 *__restrict__ lo2, int p,
                                            double x0, double y0, double side, double2 &dw, double2 &phi, double2 &dphi)
{
    dw = phi = dphi = make_double2(0.0, 0.0);
    double2 va, da, vb, db;
    const int e1 = w_off[A + 1];
    int e = w_off[A], D = 0;
    int4 cd = make_int4(0, 0, 0, 0);
    if (e < e1) {
        D = w_idx[e];
        cd = cell[D];
    }
    if (c.x >= 2) {
        const double w = ldexp(side, -c.x);
        const double2 ctr = cell_centre(x0, y0, side, c);
        const double2 xi = make_double2((z.x - ctr.x) / w, (z.y - ctr.y) / w);
        horner_pair(lo + (int64_t)A * p, lo2 + (int64_t)A * p, p, xi, va, da, vb, db);
        phi = make_double2(vb.x / w, vb.y / w);
        dphi = make_double2(db.x / (w * w), db.y / (w * w));
        dw = make_double2(da.x / (w * w), da.y / (w * w));
    }
    for (; e < e1; ++e) {
        const double w = ldexp(side, -cd.x);
        const double2 ctr = cell_centre(x0, y0, side, cd);
        const double2 *const a = mp + (int64_t)D * p, *const b = mp2 + (int64_t)D * p;
        if (e + 1 < e1) {
            D = w_idx[e + 1];
            cd = cell[D];
        }
        const double rw = 1.0 / w;
        const double2 x = cinv(make_double2((z.x - ctr.x) * rw, (z.y - ctr.y) * rw));
        horner_pair(a, b, p, x, va, da, vb, db);
        const double2 xw = make_double2(x.x * rw, x.y * rw);
        const double2 x2 = cmul<double>(xw, xw);
        phi = cmac<double>(phi, xw, vb);
        const double2 sq = cmul<double>(x2, cmac<double>(vb, x, db)), sc = cmul<double>(x2, cmac<double>(va, x, da));
        dphi = make_double2(dphi.x - sq.x, dphi.y - sq.y);
        dw = make_double2(dw.x - sc.x, dw.y - sc.y);
    }
}

// Adjoint finalize: the near sums (record units: Phi scaled by alpha, A and B by
// alpha^2 / (2 pi), as for the uniform tree) combined with the far parts:
//   dL/dGamma = -Im(Phi_near + Phi_far)/(2 pi),
//   dL/dx_eval = Re(q (A + B + W')), dL/dy_eval = -Im(q (A - B + W'))   (B imaginary),
//   dL/dx_src = -Re(c (At + Bt)),     dL/dy_src = Im(c (At - Bt)),  At = near + Phi'.
template <bool SRC>
__global__ __launch_bounds__(256) void at_finalize_backward_kernel(
    int n, const int *__restrict__ perm, const int *__restrict__ leaf_of, const int4 *__restrict__ cell,
    const double2 *__restrict__ xy, const int *__restrict__ w_off, const int *__restrict__ w_idx,
    const double2 *__restrict__ mp, const double2 *__restrict__ lo, const double2 *__restrict__ mp2,
    const double2 *__restrict__ lo2, int p, double x0, double y0, double side, const double4 *__restrict__ near_pa,
    const double4 *__restrict__ near_src, const double2 *__restrict__ adj,
    const double *__restrict__ gamma, double alpha, double lambda, AdjointOut out)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    // the per-particle loads first, in flight during the far-field work
    const int64_t o = perm[i];
    const double4 a = near_pa[i];
    const int A = leaf_of[i];
    const int4 c = cell[A];
    const double2 z = xy[i];
    double2 dw, phi, dphi;
    far_adjoint(A, c, z, w_off, w_idx, cell, mp, lo, mp2, lo2, p, x0, y0, side, dw, phi, dphi);
    const double ka = alpha * alpha * kInv2Pi;
    const double Ar = ka * (-2.0 * a.z), Ai = -ka * a.y;
    const double Bi = -ka * lambda * a.w;
    const double g = -(alpha * a.x + phi.y) * kInv2Pi;
    double ex = 0.0, ey = 0.0, sx = 0.0, sy = 0.0;
    if (out.dxe || out.dxy) {
        const double2 q = adj[i];
        const double d1r = Ar + dw.x, d1i = Ai + Bi + dw.y;
        const double d2r = Ar + dw.x, d2i = Ai - Bi + dw.y;
        ex = q.x * d1r - q.y * d1i;
        ey = -(q.x * d2i + q.y * d2r);
    }
    if constexpr (SRC) {
        const double4 ns = near_src[i];
        const double a2 = alpha * alpha;
        const double atr = a2 * ns.x + dphi.x, ati = a2 * ns.y + dphi.y;
        const double btr = a2 * lambda * ns.z, bti = a2 * lambda * ns.w;
        const double G = gamma[i] * kInv2Pi;  // c = -i G: Re(c w) = G Im w, Im(c w) = -G Re w
        sx = -G * (ati + bti);
        sy = -G * (atr - btr);
    }
    store_adjoint(out, o, g, ex, ey, sx, sy);
}

// Adjoint finalize of the pair force: the near sums combined, the far parts as above.
__global__ __launch_bounds__(256) void at_finalize_force_kernel(
    int n, const int *__restrict__ perm, const int *__restrict__ leaf_of, const int4 *__restrict__ cell,
    const double2 *__restrict__ xy, const int *__restrict__ w_off, const int *__restrict__ w_idx,
    const double2 *__restrict__ mp, const double2 *__restrict__ lo, const double2 *__restrict__ mp2,
    const double2 *__restrict__ lo2, int p, double x0, double y0, double side, const ForceNear near,
    const double2 *__restrict__ adj, const double *__restrict__ gamma, double alpha, AdjointOut out)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    // the per-particle loads first, in flight during the far-field work
    const int64_t o = perm[i];
    const int A = leaf_of[i];
    const int4 c = cell[A];
    const double2 z = xy[i], q = adj[i];
    const double G = gamma[i] * kInv2Pi;
    const int m = near.mask[A];
    const double2 nr = near_from_slots<double>(i, n, m, near.near, (const double2 *)near.slots, alpha * alpha * kInv2Pi);
    double nphi = 0.0;
    if (out.dg) nphi = alpha * phi_from_slots<double>(i, n, m, near.phi, (const double *)near.phi_slots);
    double2 dw, phi, dphi;
    far_adjoint(A, c, z, w_off, w_idx, cell, mp, lo, mp2, lo2, p, x0, y0, side, dw, phi, dphi);
    store_adjoint(out, o, -(nphi + phi.y) * kInv2Pi, nr.x + (q.x * dw.x - q.y * dw.y),
                  nr.y - (q.x * dw.y + q.y * dw.x), -G * dphi.y, -G * dphi.x);
}

inline unsigned blocks(int64_t work, int per) { return (unsigned)((work + per - 1) / per); }

}  // namespace

void launch_atree_pack(const AtreeCall &c, const double *gamma, hipStream_t s)
{
    const fmm_atree *t = c.t;
    const int n = (int)t->n;
    const bool direct = direct_rows(n, kForwardRow);
    if (!direct) launch_stage_rows(n, t->stage_shift, t->d.gpos1, gamma, t->d.st1, s);
    const int *idx = direct ? t->d.perm : t->d.gpos2;
    const double *rows = direct ? gamma : t->d.st1;
    const unsigned g = xcd_grid(n, 256, kXcds);
    if (c.is_double)
        at_pack_kernel<double><<<g, 256, 0, s>>>(n, kXcds, idx, rows, (double *)t->wsp->gam, t->wsp->gamma);
    else
        at_pack_kernel<float><<<g, 256, 0, s>>>(n, kXcds, idx, rows, (float *)t->wsp->gam, t->wsp->gamma);
}

void launch_atree_coords(const fmm_atree *t, int is_double, void *pos, hipStream_t s)
{
    const int n = (int)t->n;
    if (is_double)
        at_coords_kernel<double><<<blocks(n, 256), 256, 0, s>>>(n, t->d.leaf_of, t->d.cell, t->d.xy, t->x0, t->y0,
                                                                t->side, (double2 *)pos);
    else
        at_coords_kernel<float><<<blocks(n, 256), 256, 0, s>>>(n, t->d.leaf_of, t->d.cell, t->d.xy, t->x0, t->y0,
                                                               t->side, (float2 *)pos);
}

// Split cells of a level up to which three levels are taken in one launch: 800001 clustered
// particles (mixed) 0.447 ms level by level, 0.401 with 512, 0.390 with 2048 and 8192 cells;
// 3000001 with their rebuild 3.68 ms, 3.70, 3.68 and 3.72.
constexpr int kSubtreeCells = 2048;

void launch_atree_far(const AtreeCall &c, hipStream_t s, bool both)
{
    const fmm_atree *t = c.t;
    const int deepest = (int)t->sizes[6];
    if (deepest < 2) return;
    const int p = c.p;
    const AtreeWs &w = *t->wsp;
    const unsigned sets = both ? 2 : 1;
    if (t->np2m > 0) {
        // 16 lanes per leaf, four leaves per wavefront
        const int np = (int)t->np2m;
        auto k = p <= 16 ? at_p2m_kernel<16, 16> : at_p2m_kernel<32, 16>;
        k<<<dim3(blocks(np, 4), sets), 64, 0, s>>>(t->d.p2m_cells, np, t->d.cell, t->d.range, t->d.xy, w.gamma, nullptr,
                                                   t->x0, t->y0, t->side, p, w.mp, w.adj, w.mp2);
    }
    TransArgs a{};
    a.p = p;
    a.no_lds = c.near_occ > 0;
    a.entries = c.tabs->mfma_entries;
    a.tab = c.tabs->mfma_d;
    a.zero = c.tabs->zero_row;
    a.first = t->level_off[2];
    a.child = t->d.child;
    a.parent = t->d.parent;
    a.vslot = t->d.vslot;
    a.x_off = t->d.x_off;
    SubtreeArgs st{};
    st.p = p;
    st.deepest = deepest;
    st.tab = c.tabs->mfma_d;
    st.child = t->d.child;
    st.zero = c.tabs->zero_row;
    // three levels from `base` on in one launch where a workgroup per split cell of `base` is
    // not many more than fit at once
    auto subtree = [&](int base, bool up) {
        const int n = t->inner_off[base + 1] - t->inner_off[base];
        if (n > kSubtreeCells) return false;
        st.base = base;
        st.rows = (double *)(up ? w.mp : w.lo);
        st.rows2 = both ? (double *)(up ? w.mp2 : w.lo2) : nullptr;
        st.cells = t->d.inner + t->inner_off[base];
        st.ncells = n;
        if (n > 0) launch_subtree(st, up, s);
        return true;
    };
    // stage 5 upward
    a.targets = t->d.inner;
    a.src = a.out = w.mp;
    if (both) a.src2 = a.out2 = w.mp2;
    a.nseg = 1;
    for (int l = deepest - 1; l >= 2; --l) {
        if (l >= 3) {
            st.deepest = l + 1;
            const int base = l >= 4 ? l - 2 : 2;
            if (subtree(base, true)) {
                l = base;
                continue;
            }
        }
        a.seg[0] = TransSeg{0, t->inner_off[l], t->inner_off[l + 1] - t->inner_off[l], l};
        launch_trans64(a, Trans::M2M, true, s);
    }
    const int cnt = t->level_off[deepest + 1] - a.first;
    if (cnt <= 0) return;
    // P2L into the locals of the cells with an X list, then the M2L from V of every level
    // added to them, then the L2L level by level downward
    if (t->sizes[5] > 0) {  // |X|
        auto k = p <= 16 ? at_p2l_kernel<16, 16> : at_p2l_kernel<32, 16>;
        k<<<dim3(blocks(cnt, 4), sets), 64, 0, s>>>(a.first, cnt, t->d.cell, t->d.x_off, t->d.x_idx, t->d.range, t->d.xy,
                                                    w.gamma, nullptr, t->x0, t->y0, t->side, p, w.lo, w.adj, w.lo2);
    }
    a.targets = t->d.m2l_targets;
    a.out = w.lo;
    if (both) a.out2 = w.lo2;
    auto level_segs = [&](int l0, int l1) {
        a.nseg = 0;
        for (int l = l0; l <= l1; ++l)
            for (int k = 0; k < 4; ++k) {
                const int *off = &t->m2l_seg_off[4 * (l - 2) + k];
                a.seg[a.nseg++] = TransSeg{0, off[0], off[1] - off[0], l};
            }
    };
    level_segs(2, deepest);
    launch_trans64(a, Trans::M2L, true, s);
    a.src = w.lo;
    if (both) a.src2 = w.lo2;
    for (int l = 3; l <= deepest; ++l) {
        st.deepest = std::min(deepest, l + 2);
        if (l < deepest && subtree(l - 1, false)) {
            l += 2;
            continue;
        }
        level_segs(l, l);
        launch_trans64(a, Trans::L2L, true, s);
    }
}

namespace {

// Occupancy cap: each near-field workgroup (one wavefront) reserves LDS so that at most near_occ
// of them fit on a SIMD (160 KiB per CU, 4 SIMDs); the far chain on the other stream takes the
// wavefront slots left over.
size_t near_lds_reserve(const AtreeCall &c, size_t static_bytes)
{
    const size_t per_wave = c.near_occ > 0 ? (size_t)160 * 1024 / (4 * (size_t)c.near_occ) : 0;
    return per_wave > static_bytes ? per_wave - static_bytes : 0;
}

}  // namespace

void launch_atree_near(const AtreeCall &c, hipStream_t s)
{
    const fmm_atree *t = c.t;
    if (t->nwork == 0) return;
    const double scale = c.alpha * kInv2Pi;
    // exponent at which 1 - e rounds to 1: FP32 base 2 at 26, FP64 base e at 37.5, one
    // unit of margin for the rounding of the records and the boxes
    const double cut = c.is_double ? 39.0 : 27.0;
    const size_t dyn = near_lds_reserve(c, 256 * (c.is_double ? sizeof(double4) : sizeof(float4)));
    if (c.is_double)
        at_near_kernel<double><<<(unsigned)t->nwork, 64, dyn, s>>>(
            t->d.work, t->d.cell, t->d.range, t->d.u_off, t->d.u_idx, t->d.tile_start, t->d.tile_box,
            t->d.leaf_start, t->d.leaf_tile, t->d.tile_box_leaf, (const double2 *)t->d_pos[1],
            (const double *)t->wsp->gam, t->x0, t->y0, t->side,
            c.alpha, cut, scale, t->dense_leaf, t->n, t->wsp->near, (double2 *)t->wsp->slots);
    else
        at_near_kernel<float><<<(unsigned)t->nwork, 64, dyn, s>>>(
            t->d.work, t->d.cell, t->d.range, t->d.u_off, t->d.u_idx, t->d.tile_start, t->d.tile_box,
            t->d.leaf_start, t->d.leaf_tile, t->d.tile_box_leaf, (const float2 *)t->d_pos[0],
            (const float *)t->wsp->gam, t->x0, t->y0, t->side,
            c.alpha, cut, scale, t->dense_leaf, t->n, t->wsp->near, (float2 *)t->wsp->slots);
}

void launch_atree_finalize(const AtreeCall &c, double *uv, double *uv_near, double *uv_far, const double *base,
                           double h, hipStream_t s)
{
    const fmm_atree *t = c.t;
    const int n = (int)t->n;
    const double scale = c.alpha * kInv2Pi;
    // uv alone: the totals go to the staging array (n double2), then to user order:
    // through the staging windows once the output fills the last-level cache, else in
    // sorted order and scattered; small outputs directly
    double2 *staged = uv && !uv_near && !uv_far && !direct_rows(n, kForwardRow) ? t->wsp->stage : nullptr;
    const bool windowed = staged && outputs_windowed(n, sizeof(double2));
    const int *gp = windowed ? t->d.gpos2 : nullptr;
    double *uv_direct = staged ? nullptr : uv;
    const unsigned g = xcd_grid(n, 256, kXcds);
    if (c.is_double)
        at_finalize_kernel<double><<<g, 256, 0, s>>>(
            n, t->d.perm, t->d.leaf_of, t->d.cell, t->d.xy, t->d.w_off, t->d.w_idx, t->wsp->mp, t->wsp->lo, c.p, t->x0,
            t->y0, t->side, t->wsp->near, t->d.mask, (const double2 *)t->wsp->slots, scale, uv_direct, uv_near, uv_far,
            staged, gp, kXcds, base, h);
    else
        at_finalize_kernel<float><<<g, 256, 0, s>>>(
            n, t->d.perm, t->d.leaf_of, t->d.cell, t->d.xy, t->d.w_off, t->d.w_idx, t->wsp->mp, t->wsp->lo, c.p, t->x0,
            t->y0, t->side, t->wsp->near, t->d.mask, (const float2 *)t->wsp->slots, scale, uv_direct, uv_near, uv_far,
            staged, gp, kXcds, base, h);
    if (windowed) launch_gather_rows(n, t->d.gpos1, staged, uv, base, h, s);
    else if (staged) scatter_rows_kernel<<<blocks(n, 256), 256, 0, s>>>(n, t->d.perm, staged, uv, base, h);
}

void launch_atree_pack_adjoint(const AtreeCall &c, const double *dl_duv, double scale, hipStream_t s)
{
    const fmm_atree *t = c.t;
    const int n = (int)t->n;
    // the forward's near-field array (n double2) is free during the adjoint: the staging
    double2 *st = t->wsp->near;
    const bool direct = direct_rows(n, kAdjointRow);
    if (!direct) launch_stage_rows2(n, t->stage_shift, t->d.gpos1, (const double2 *)dl_duv, st, s);
    const int *idx = direct ? t->d.perm : t->d.gpos2;
    const double2 *rows = direct ? (const double2 *)dl_duv : st;
    const unsigned g = xcd_grid(n, 256, kXcds);
    if (c.is_double)
        at_pack_adjoint_kernel<double><<<g, 256, 0, s>>>(n, kXcds, idx, rows, scale, t->wsp->adj,
                                                         (double2 *)t->wsp->qt);
    else
        at_pack_adjoint_kernel<float><<<g, 256, 0, s>>>(n, kXcds, idx, rows, scale, t->wsp->adj,
                                                        (float2 *)t->wsp->qt);
}

void launch_atree_backward_near(const AtreeCall &c, bool src, hipStream_t s)
{
    const fmm_atree *t = c.t;
    if (t->nbwd_units <= 0) return;
    const double cut = c.is_double ? 39.0 : 27.0;  // as for the forward near field
    const unsigned g = (unsigned)t->nbwd_units;
    const AtreeDev &d = t->d;
    const AtreeWs &w = *t->wsp;
    if (c.is_double) {
        auto k = src ? at_backward_kernel<double, true> : at_backward_kernel<double, false>;
        k<<<g, 64, 0, s>>>(d.bwd_units, d.cell, d.range, d.u_off, d.u_idx, d.tile_start, d.tile_box,
                           (const double2 *)t->d_pos[1], (const double *)w.gam, (const double2 *)w.qt, t->x0,
                           t->y0, t->side, c.alpha, cut, 1.0,
                           w.pa, src ? w.psrc : nullptr);
    } else {
        auto k = src ? at_backward_kernel<float, true> : at_backward_kernel<float, false>;
        k<<<g, 64, 0, s>>>(d.bwd_units, d.cell, d.range, d.u_off, d.u_idx, d.tile_start, d.tile_box,
                           (const float2 *)t->d_pos[0], (const float *)w.gam, (const float2 *)w.qt, t->x0,
                           t->y0, t->side, c.alpha, cut,
                           0.69314718055994530942f, w.pa, src ? w.psrc : nullptr);
    }
}

namespace {

template <int KIND> void force_launch(const AtreeCall &c, const ForceNear &near, hipStream_t s)
{
    const fmm_atree *t = c.t;
    const AtreeDev &d = t->d;
    at_force_kernel<KIND><<<(unsigned)t->nwork, 64, near_lds_reserve(c, sizeof(NearLds<double, KIND>)), s>>>(
        d.work, d.cell, d.range, d.u_off, d.u_idx, d.tile_start, d.tile_box, d.leaf_start, d.leaf_tile,
        d.tile_box_leaf,
        SoaRec<double>{(const double2 *)t->d_pos[1], (const double *)t->wsp->gam, c.alpha, (const double2 *)t->wsp->qt},
        t->x0, t->y0, t->side, c.alpha, 39.0, t->dense_leaf, t->n, near.near, near.phi, (double2 *)near.slots,
        (double *)near.phi_slots);  // (the cut as for the forward near field)
}

}  // namespace

void launch_atree_force(const AtreeCall &c, const ForceNear &near, hipStream_t s)
{
    if (c.t->nwork == 0) return;
    auto k = near.phi ? force_launch<kForcePhi> : force_launch<kForce>;
    k(c, near, s);
}

void launch_atree_finalize_force(const AtreeCall &c, const ForceNear &near, const AdjointOut &out, hipStream_t s)
{
    const fmm_atree *t = c.t;
    const int n = (int)t->n;
    const AtreeDev &d = t->d;
    const AtreeWs &w = *t->wsp;
    at_finalize_force_kernel<<<blocks(n, 256), 256, 0, s>>>(
        n, d.perm, d.leaf_of, d.cell, d.xy, d.w_off, d.w_idx, w.mp, w.lo, w.mp2, w.lo2,
                                     c.p, t->x0, t->y0, t->side, near, w.adj, w.gamma, c.alpha, out);
}

void launch_atree_finalize_backward(const AtreeCall &c, const AdjointOut &out, hipStream_t s)
{
    const fmm_atree *t = c.t;
    const int n = (int)t->n;
    const double lambda = c.is_double ? 1.0 : 0.69314718055994530942;
    const AtreeDev &d = t->d;
    const AtreeWs &w = *t->wsp;
    auto k = (out.dxs || out.dxy) ? at_finalize_backward_kernel<true> : at_finalize_backward_kernel<false>;
    k<<<blocks(n, 256), 256, 0, s>>>(n, d.perm, d.leaf_of, d.cell, d.xy, d.w_off, d.w_idx, w.mp, w.lo, w.mp2, w.lo2,
                                     c.p, t->x0, t->y0, t->side, w.pa, w.psrc, w.adj, w.gamma, c.alpha, lambda,
                                     out);
}

}  // namespace fmm
