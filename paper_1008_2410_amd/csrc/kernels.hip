// gfx950 kernels of the FMM evaluation phase (stages 4-10 of Fig. fmmStages of
// Knepley, arXiv:1008.2410) and their host launchers.
//
// Conventions (shared with api.cpp, host_tree.cpp and tree_build.hip):
//  - Particles are in leaf-Morton order ("sorted"); d_perm maps a sorted slot to the
//    user index, d_leaf_of to its leaf.
//  - Complex charge c_j = -i Gamma_j / (2 pi) (the factor of the multipole
//    coefficients, section "Complexity Estimates"); conjugate velocity W = u - i v.
//  - Expansions are radius-scaled so every translation operator is level independent:
//    multipole a_m / w^m, local b_l w^(l+1), with w the cell width of the level.
//  - Complex numbers are interleaved (re, im) float2 / double2.
#include "fmm_internal.h"
#include "device_common.h"
#include "translate.h"

#include <algorithm>
#include <climits>
#include <cmath>
#include <mutex>
#include <type_traits>

namespace fmm {
namespace {

// ---------------------------------------------------------------------------------
// Circulations from user order into tree order in two passes.  The user order is
// arbitrary (a random shuffle in the benchmark), so a direct gather makes one random
// memory access per element.  Instead, with buckets of 2^S consecutive sorted slots:
//   pass 1 (stage_in_kernel) reads a contiguous chunk of user indices, sorts it in LDS
//          by bucket and writes each bucket's elements as one run into that bucket's
//          segment of a staging array (inside a bucket, slots follow user index, so a
//          chunk's elements of one bucket are one contiguous run);
//   pass 2 (in pack_kernel) walks the sorted slots and gathers from the current
//          bucket's segment, a window small enough to stay in one XCD's L2.
// gpos1[user index] = staging slot; gpos2[sorted slot] = staging slot of its user index.
// S is chosen with the tree so that there are at most kStageBuckets.  Blocks are remapped
// so that each XCD (workgroups are dealt to XCDs round-robin) walks one contiguous index
// range, which keeps its live windows few.
// ---------------------------------------------------------------------------------
constexpr int kStageE = 4;  // elements per thread in pass 1 (chunk of 1024)

template <typename V>
__global__ __launch_bounds__(256) void stage_in_kernel(int n, int shift, int nxcd, const int *__restrict__ gpos1,
                                                        const V *__restrict__ src, V *__restrict__ st)
{
    constexpr int C = 256 * kStageE;
    __shared__ int cnt[kStageBuckets], lo[kStageBuckets], off[kStageBuckets];
    __shared__ V val[C];
    __shared__ int dst[C];
    const int t = threadIdx.x;
    const int nb = ((n - 1) >> shift) + 1;  // buckets in use, <= kStageBuckets by the choice of shift
    for (int b = t; b < nb; b += 256) {
        cnt[b] = 0;
        lo[b] = INT_MAX;
    }
    __syncthreads();
    const int64_t k0 = (int64_t)xcd_block(nxcd) * C;
    int q[kStageE];
    V v[kStageE];
#pragma unroll
    for (int e = 0; e < kStageE; ++e) {
        const int64_t k = k0 + e * 256 + t;
        q[e] = -1;
        v[e] = V{};
        if (k < n) {
            q[e] = gpos1[k];
            v[e] = src[k];
            const int bk = q[e] >> shift;
            atomicAdd(&cnt[bk], 1);
            atomicMin(&lo[bk], q[e]);
        }
    }
    __syncthreads();
    if (t < 64) {  // exclusive scan of the bucket counts by one wavefront, a run of buckets per lane
        const int per = (nb + 63) / 64;
        const int b0 = t * per, b1 = min(b0 + per, nb);
        int sum = 0;
        for (int b = b0; b < b1; ++b) sum += cnt[b];
        int incl = sum;
        for (int d = 1; d < 64; d <<= 1) {
            const int o = __shfl_up(incl, d);
            if (t >= d) incl += o;
        }
        int run = incl - sum;
        for (int b = b0; b < b1; ++b) {
            off[b] = run;
            run += cnt[b];
        }
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < kStageE; ++e)
        if (q[e] >= 0) {
            const int bk = q[e] >> shift;
            const int slot = off[bk] + (q[e] - lo[bk]);  // < C: the bucket's run is contiguous
            val[slot] = v[e];
            dst[slot] = q[e];
        }
    __syncthreads();
    const int m = (int)min((int64_t)C, (int64_t)n - k0);
    for (int j = t; j < m; j += 256) st[dst[j]] = val[j];
}

// Pass 2 of the user-to-tree permutation: the circulation of sorted particle i, read from
// the staging array at gpos2[i] and rounded to the near field's precision (the near-field
// records' Gamma; the positions of the records are the tree's, in leaf units).
template <typename T>
__global__ __launch_bounds__(256) void pack_kernel(int n, int nxcd, const int *__restrict__ gpos2,
                                                    const double *__restrict__ gamma_st, T *__restrict__ gam)
{
    const int i = xcd_block(nxcd) * blockDim.x + threadIdx.x;
    if (i >= n) return;
    gam[i] = (T)gamma_st[gpos2[i]];
}

// Leaf-unit coordinates xi = (z - c_leaf)/w_L of the sorted particles (the tree's, made once
// per precision): the near-field records are xi scaled by alpha w_L on load, and L2P and
// P2M evaluate their series at xi.
template <typename T>
__global__ __launch_bounds__(256) void leaf_coords_kernel(int n, const int *__restrict__ leaf_of,
                                                           const double2 *__restrict__ xy, double x0, double y0,
                                                           double w, c2<T> *__restrict__ pos)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const uint32_t leaf = (uint32_t)leaf_of[i];
    const double cx = x0 + (morton_x(leaf) + 0.5) * w;
    const double cy = y0 + (morton_y(leaf) + 0.5) * w;
    const double2 z = xy[i];
    pos[i] = mk<T>((T)((z.x - cx) / w), (T)((z.y - cy) / w));
}


// ---------------------------------------------------------------------------------
// Stage 9, P2P (near field), target-centric: every pair is evaluated from the target's
// end, so no output is shared between work-items (the paper computes each pair from
// both ends to avoid memory contention).  One wavefront per work unit
// {leaf T, first target, count nt <= 64, log2 TP}: lane = k*TP + t handles target t
// and, of every 64-source tile of the 3x3 leaf neighbourhood, the sources k, k+K, ...
// (K = 64/TP), so sparse leaves still fill the wavefront.
//
// Source tiles are the 64-particle, leaf-aligned chunks of the sorted order (particles
// inside a leaf are ordered by a finer Morton key, so a tile is spatially compact).
// Each tile is staged in LDS (one coalesced load, then broadcast reads) and tested
// against the bounding box of the target chunk: when every pair of the tile has
// s >= cut, 1 - exp(-s) rounds to exactly 1 in T and the exponential is skipped --
// the result is bit-identical to evaluating it.
// Per-leaf partial sums are kept in T and folded into FP64; the K partial sums of a
// target are combined by lane shuffles.
//   velocity u = -(alpha/2pi) sum Gamma g dY/s,  v = (alpha/2pi) sum Gamma g dX/s
// ---------------------------------------------------------------------------------

template <typename T>
__device__ __forceinline__ void p2p_forward_unit(const int4 u, rec_t<T> *tile, const SoaRec<T> &rec,
                                                 const int *__restrict__ leaf_start,
                                                 const int *__restrict__ tile_start,
                                                 const float4 *__restrict__ tile_box, int nside, T step,
                                                 float cut_leaf2, double scale, int dense,
                                                 double2 *__restrict__ near)
{
    const int lane = threadIdx.x;
    const int logtp = u.w & 15;
    const bool skip_dense = (u.w >> 4) != 0;  // pairs with dense leaves go to the mutual form
    const int ix = (int)morton_x((uint32_t)u.x), iy = (int)morton_y((uint32_t)u.x);
    // lane d < 9: the range of neighbour leaf d
    int s0 = 0, len = 0, ddx = 0, ddy = 0;
    uint32_t S = 0;
    if (lane < 9) {
        ddx = lane % 3 - 1;
        ddy = lane / 3 - 1;
        const int nx = ix + ddx, ny = iy + ddy;
        if (nx >= 0 && ny >= 0 && nx < nside && ny < nside) {
            S = morton_encode((uint32_t)nx, (uint32_t)ny);
            s0 = leaf_start[S];
            len = leaf_start[S + 1] - s0;
            if (skip_dense && len >= dense) len = 0;
        }
    }
    if (!__any(len > 64)) {  // every source leaf is one tile
        const UnitLanes ul(lane, u.z, logtp);
        const int i = u.y + min(ul.t, u.z - 1);
        const rec_t<T> ri = rec(i);
        bool far = false;
        if (cut_leaf2 < 8.0f && len > 0) {  // (no tile of the neighbourhood is sqrt(8) leaves away)
            const float4 tbox = tile_box[tile_start[u.x] + ((u.y - leaf_start[u.x]) >> 6)];
            far = box_gap2(tbox, (float)-ddx, (float)-ddy, tile_box[tile_start[S]]) >= cut_leaf2;
        }
        const T ox = (T)ddx * step, oy = (T)ddy * step;
        double au = 0.0, av = 0.0;
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
        source_batches<16>(far ? 0 : len, stage, [&](int count) {
            T fu = 0, fv = 0;
            p2p_batch<T, false>(tile, count, ul.k, ul.K, ri.x, ri.y, fu, fv);
            au += (double)fu;
            av += (double)fv;
        });
        if (__any(far))
            source_batches<16>(far ? len : 0, stage, [&](int count) {
                T fu = 0, fv = 0;
                p2p_batch<T, true>(tile, count, ul.k, ul.K, ri.x, ri.y, fu, fv);
                au += (double)fu;
                av += (double)fv;
            });
        au = ul.reduce(au);
        av = ul.reduce(av);
        if (lane < u.z) near[i] = make_double2(-scale * au, scale * av);
        return;
    }
    const int tp = 1 << logtp;
    const int t = lane & (tp - 1);
    const int k = lane >> logtp;
    const int i = u.y + min(t, u.z - 1);
    const rec_t<T> ri = rec(i);
    const float4 tbox = tile_box[tile_start[u.x] + ((u.y - leaf_start[u.x]) >> 6)];
    double au = 0.0, av = 0.0;
    for (int dy = -1; dy <= 1; ++dy) {
        const int ny = iy + dy;
        if (ny < 0 || ny >= nside) continue;
        for (int dx = -1; dx <= 1; ++dx) {
            const int nx = ix + dx;
            if (nx < 0 || nx >= nside) continue;
            const uint32_t S = morton_encode((uint32_t)nx, (uint32_t)ny);
            const int s0 = leaf_start[S], s1 = leaf_start[S + 1];
            if (skip_dense && s1 - s0 >= dense) continue;
            // target relative to the centre of leaf S: z_i - c_S = (z_i - c_T) + (c_T - c_S)
            const T tx = ri.x - (T)dx * step;
            const T ty = ri.y - (T)dy * step;
            T fu = 0, fv = 0;
            int tt = tile_start[S];
            for (int base = s0; base < s1; base += 64, ++tt) {
                const int len = min(64, s1 - base);
                __syncthreads();
                if (lane < len) tile[lane] = rec(base + lane);
                const bool far = box_gap2(tbox, (float)-dx, (float)-dy, tile_box[tt]) >= cut_leaf2;
                __syncthreads();
                switch (logtp) {
                case 6: p2p_tile_any<T, 1>(tile, len, k, tx, ty, fu, fv, far); break;
                case 5: p2p_tile_any<T, 2>(tile, len, k, tx, ty, fu, fv, far); break;
                case 4: p2p_tile_any<T, 4>(tile, len, k, tx, ty, fu, fv, far); break;
                case 3: p2p_tile_any<T, 8>(tile, len, k, tx, ty, fu, fv, far); break;
                case 2: p2p_tile_any<T, 16>(tile, len, k, tx, ty, fu, fv, far); break;
                case 1: p2p_tile_any<T, 32>(tile, len, k, tx, ty, fu, fv, far); break;
                default: p2p_tile_any<T, 64>(tile, len, k, tx, ty, fu, fv, far); break;
                }
            }
            au += (double)fu;
            av += (double)fv;
        }
    }
    for (int o = tp; o < 64; o <<= 1) {
        au += __shfl_xor(au, o);
        av += __shfl_xor(av, o);
    }
    if (k == 0 && t < u.z) near[i] = make_double2(-scale * au, scale * av);
}

// Near-field grid (stage 9): one list of work entries, each one wavefront's work:
//   mutual items {S, R, d_S | d_R << 4, kMutualItem}, d_S = direction of R seen from S
//   and d_R = 8 - d_S, writing the slots (9 x n sums (dY, dX) in the records'
//   precision, unscaled);
//   target-centric units {leaf, first, count, log2 TP | 16 if dense neighbours are
//   skipped}, writing near.
// The list is sorted by estimated cost, heaviest first, and launched as one workgroup
// per entry: the hardware dispatcher hands them out in order.  Each entry writes only
// its own outputs, so the result does not depend on which wavefront takes which entry.

template <typename T>
__global__ __launch_bounds__(64, sizeof(T) == 4 ? 8 : 5) void p2p_near_kernel(
    const int4 *__restrict__ work, const c2<T> *__restrict__ pos, const T *__restrict__ gam,
    const int *__restrict__ leaf_start, const int *__restrict__ tile_start, const float4 *__restrict__ tile_box,
    int nside, T step, float cut_leaf2, double scale, int dense, int64_t n, double2 *__restrict__ near,
    c2<T> *__restrict__ slots, const MutualParts parts)
{
    __shared__ NearLds<T, kVelocity> lds;
    const SoaRec<T> rec{pos, gam, step};
    const int4 u = work[blockIdx.x];
    if (u.w & kMutualItem)
        mutual_item<kVelocity>(u, lds, rec, MutualTree{leaf_start, tile_start, tile_box, cut_leaf2, 0.0f}, parts,
                               step, n, slots, (T *)nullptr);
    else
        p2p_forward_unit<T>(u, lds.a, rec, leaf_start, tile_start, tile_box, nside, step, cut_leaf2, scale, dense,
                            near);
}

// The target's own factors in FP64, for the FP32 units: adjoint charges and circulations, and the
// power of two the FP32 charges carry.
struct ForceTargets {
    const double2 *__restrict__ adj;
    GammaRows gamma;
    const double *__restrict__ qscale;
};

// The adjoint's target-centric unit over the pair force: the forward's, with every source
// leaf in the concatenation (a leaf of one tile beyond the cut skips the exponential).
template <typename T, int KIND>
__device__ __forceinline__ void p2p_force_unit(const int4 u, rec_t<T> *tile, T *qtile, const SoaRec<T> &rec,
                                               const ForceTargets &own, const MutualTree &mt, int nside, T step,
                                               double scale, int dense, double2 *__restrict__ near,
                                               double *__restrict__ near_phi)
{
    // FP64: the sums of the pair force; FP32: the separate sums (see p2p_force_kernel)
    constexpr int NS = sizeof(T) == 4 ? 8 : kSums<KIND>;
    const int lane = threadIdx.x;
    const bool skip_dense = (u.w >> 4) != 0;  // pairs with dense leaves go to the mutual form
    const int ix = (int)morton_x((uint32_t)u.x), iy = (int)morton_y((uint32_t)u.x);
    // lane d < 9: the range of neighbour leaf d
    int s0 = 0, len = 0, ddx = 0, ddy = 0;
    bool far = false;
    if (lane < 9) {
        ddx = lane % 3 - 1;
        ddy = lane / 3 - 1;
        const int nx = ix + ddx, ny = iy + ddy;
        if (nx >= 0 && ny >= 0 && nx < nside && ny < nside) {
            const uint32_t S = morton_encode((uint32_t)nx, (uint32_t)ny);
            s0 = mt.leaf_start[S];
            len = mt.leaf_start[S + 1] - s0;
            if (skip_dense && len >= dense) len = 0;
            if (mt.cut_leaf2 < 8.0f && len > 0 && len <= 64) {
                const float4 tbox = mt.tile_box[mt.tile_start[u.x] + ((u.y - mt.leaf_start[u.x]) >> 6)];
                far = box_gap2(tbox, (float)-ddx, (float)-ddy, mt.tile_box[mt.tile_start[S]]) >= mt.cut_leaf2;
            }
        }
    }
    const UnitLanes ul(lane, u.z, u.w & 15);
    const int i = u.y + min(ul.t, u.z - 1);
    T tiqy;
    const rec_t<T> ti = load_rec<KIND>(rec, i, tiqy);
    const T ox = (T)ddx * step, oy = (T)ddy * step;
    double sum[NS] = {};
    auto stage = [&](int e, int j) {
        const int from = __shfl(s0, e);
        const T sx = __shfl(ox, e), sy = __shfl(oy, e);
        stage_source<KIND>(tile, qtile, rec, j >= 0 ? from + j : -1, sx, sy);
    };
    source_batches<16>(far ? 0 : len, stage, [&](int count) {
        T f[NS] = {};
        if constexpr (sizeof(T) == 4) force_sums_batch<T, false>(tile, qtile, count, ul.k, ul.K, ti.x, ti.y, f);
        else force_batch<T, KIND, 0>(tile, qtile, count, ul.k, ul.K, ti, tiqy, f);
        for (int m = 0; m < NS; ++m) sum[m] += (double)f[m];
    });
    if (__any(far))
        source_batches<16>(far ? len : 0, stage, [&](int count) {
            T f[NS] = {};
            if constexpr (sizeof(T) == 4) force_sums_batch<T, true>(tile, qtile, count, ul.k, ul.K, ti.x, ti.y, f);
            else force_batch<T, KIND, 2>(tile, qtile, count, ul.k, ul.K, ti, tiqy, f);
            for (int m = 0; m < NS; ++m) sum[m] += (double)f[m];
        });
    for (int m = 0; m < NS; ++m) sum[m] = ul.reduce(sum[m]);
    if (lane >= u.z) return;
    if constexpr (sizeof(T) == 4) {
        // as finalize_backward_kernel: q (A, B) and -Gamma (At, Bt), the latter of charges that
        // carry qscale, which the sum takes on as a whole
        constexpr double lam = 0.69314718055994530942;
        const double2 q = own.adj[i];
        const double qs = *own.qscale, g = scale * own.gamma.rows[own.gamma.idx[i]];
        const double Ar = scale * (-2.0 * sum[2]), Ai = -scale * sum[1], Bi = -scale * lam * sum[3];
        near[i] = make_double2(qs * (q.x * Ar - q.y * (Ai + Bi)) - g * (sum[5] + lam * sum[7]),
                               -qs * (q.x * (Ai - Bi) + q.y * Ar) - g * (sum[4] - lam * sum[6]));
        if constexpr (KIND == kForcePhi) near_phi[i] = sum[0];
    } else {
        near[i] = make_double2(-scale * sum[0], scale * sum[1]);
        if constexpr (KIND == kForcePhi) near_phi[i] = sum[2];
    }
}

// The near-field grid of the pair force, over the forward's work list.  FP32 issues about 34
// vector operations per unordered pair (42 with the series, 41 with Phi) against 36 per ordered
// pair of the separate sums: 2^22 patch particles at depth 9, FP32, 3.6 -> 2.1 ms; 700001 at
// depth 8 in FP64 with Phi, whose exponential alone is some 25 operations, 1.2 -> 0.74 ms.
//
// The position derivative is what is left of two larger sums, so the rounding of FP32 running sums
// shows in it.  Errors of dl_dx against the FP64 call, in units of the separate sums' (uniform
// particles, sigma of 0.05 to 1 leaf, smooth and random circulations and cotangents, worst of 16):
//  - mutual items with running sums over a whole tile: 1.04 at 32 particles per leaf, 1.05 at 48, 1.07
//    at 64, 0.91 at 250; with each chunk's 16 terms added up apart 0.98, 0.97, 0.96 and 0.81 (2^20
//    uniform particles at depth 7: 0.433 -> 0.431 ms);
//  - target-centric units over the pair force 1.54 at 4 particles per leaf, 1.45 at 10, 1.40 at 16 and
//    24.  In FP32 they take the separate sums, whose terms meet the target's own FP64 factors after
//    the sums: 1.00 at each (2^20 uniform particles at depth 8: 0.373 -> 0.400 ms).
template <typename T, int KIND>
__global__ __launch_bounds__(64, sizeof(T) == 4 ? (KIND == kForcePhi ? 5 : 6) : 3) void p2p_force_kernel(
    const int4 *__restrict__ work, const SoaRec<T> rec, const ForceTargets own, const MutualTree mt, int nside, T step,
    double scale, int dense, int64_t n, double2 *__restrict__ near, double *__restrict__ near_phi,
    c2<T> *__restrict__ slots, T *__restrict__ phi_slots, const MutualParts parts)
{
    __shared__ NearLds<T, KIND> lds;
    const int4 u = work[blockIdx.x];
    if (u.w & kMutualItem) mutual_item<KIND>(u, lds, rec, mt, parts, step, n, slots, phi_slots);
    else p2p_force_unit<T, KIND>(u, lds.a, lds.qa, rec, own, mt, nside, step, scale, dense, near, near_phi);
}

// Stage 4, P2M: a_m / w^m = sum_j c_j xi_j^m, G lanes per leaf (64/G leaves per wavefront),
// each over every G-th particle.  Bound by the chain of loads before a leaf's first term (list,
// offsets, staging slot, circulation), so several leaves share a wavefront; G follows the mean
// occupancy (p2m_launch).  2^24 patch particles at depth 10, FP32: 285 us with a wavefront per
// leaf, 252 with 16 lanes, 220 with 32; 2^22 at depth 9: 77, 60 and 54.  (A wavefront per
// sparse leaf idles most lanes: 2^22 uniform particles in 2^20 leaves, 577 us.)
template <typename TR, typename TC, int PMAX, int G>
__global__ __launch_bounds__(64) void p2m_kernel(const int *__restrict__ leaves, int nleaves,
                                                  const int *__restrict__ leaf_start,
                                                  const double2 *__restrict__ xy, const c2<TC> *__restrict__ pos,
                                                  const int *__restrict__ gpos2, const double *__restrict__ gamma_st,
                                                  const typename RecScalar<TR>::type *__restrict__ gam,
                                                  const double2 *adj, double x0, double y0, double w, int p,
                                                  c2<TC> *out, int nxcd, const double2 *adj2, c2<TC> *out2)
{
    if (blockIdx.y) {  // the second set of charges
        adj = adj2;
        out = out2;
    }
    constexpr int NC = 2 * PMAX;             // partial sums per lane (re, im interleaved)
    const int lane = threadIdx.x, g = lane % G;
    // each XCD takes a contiguous run of leaves, so the staging windows its circulation
    // reads fall in stay in its own L2
    const int li = xcd_block(nxcd) * (64 / G) + lane / G;
    const bool valid = li < nleaves;  // a group past the end idles (its shuffles stay inside it)
    const uint32_t leaf = valid ? (uint32_t)leaves[li] : 0;
    const int s0 = valid ? leaf_start[leaf] : 0, s1 = valid ? leaf_start[leaf + 1] : 0;
    const double cx = x0 + (morton_x(leaf) + 0.5) * w;
    const double cy = y0 + (morton_y(leaf) + 0.5) * w;
    TC v[NC];
#pragma unroll
    for (int m = 0; m < NC; ++m) v[m] = (TC)0;
    for (int j = s0 + g; j < s1; j += G) {
        c2<TC> xi;
        if (pos) {
            xi = pos[j];  // the tree's leaf-unit coordinates, made by the same formula
        } else {
            const double2 z = xy[j];
            xi = mk<TC>((TC)((z.x - cx) / w), (TC)((z.y - cy) / w));
        }
        c2<TC> pw;
        if (adj) {
            const double2 q = adj[j];
            pw = mk<TC>((TC)q.x, (TC)q.y);
        } else {
            // the circulation as the records hold it (rounded to their precision): from the
            // gathered circulations, or from the staging array when P2M starts before them
            const double gj = gam ? (double)gam[j] : (double)(typename RecScalar<TR>::type)gamma_st[gpos2[j]];
            pw = mk<TC>(0, (TC)(-gj * kInv2Pi));
        }
#pragma unroll
        for (int m = 0; m < PMAX; ++m) {
            if (m < p) {
                v[2 * m] += pw.x;
                v[2 * m + 1] += pw.y;
                pw = cmul<TC>(pw, xi);
            }
        }
    }
    lane_halve<TC, NC, NC, G / 2>(v, lane);
    if (valid) store_halved<TC, NC, G>(v, g, 2 * p, (TC *)out + (int64_t)leaf * 2 * p);
}

// ---------------------------------------------------------------------------------
// Stages 8 + 10: L2P from the leaf's local expansion (Horner in xi = (z - c)/w_L,
// W_far = (1/w_L) sum_l b_l xi^l), plus the near field, scattered to user order:
// (u, v) = (u_near + Re W_far, v_near - Im W_far).  (A two-pass scatter through a
// staging array, as for the circulations, measured no faster for (u, v) pairs.)
// ---------------------------------------------------------------------------------
// Near field of a particle: with the mutual form (mask != NULL), the target-centric
// part (if mask bit 9 of its leaf) plus the slots d with mask bit d, in order d = 0..8.
template <typename TL, typename TS>
__global__ __launch_bounds__(256) void finalize_kernel(int n, const int *__restrict__ perm,
                                                        const int *__restrict__ leaf_of,
                                                        const double2 *__restrict__ xy,
                                                        const double2 *__restrict__ near,
                                                        const uint16_t *__restrict__ mask,
                                                        const c2<TS> *__restrict__ slots, double scale,
                                                        const c2<TL> *__restrict__ loc, const c2<TL> *__restrict__ pos,
                                                        int p, int has_far, double x0,
                                                        double y0, double w, double *__restrict__ uv,
                                                        double *__restrict__ uv_near, double *__restrict__ uv_far,
                                                        double2 *__restrict__ staged, const int *__restrict__ gpos2,
                                                        int nxcd, const double *base, double h)
{
    const int i = xcd_block(nxcd) * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int64_t o = staged ? 0 : perm[i];  // issued with the first loads
    const uint32_t leaf = (uint32_t)leaf_of[i];
    const double2 nr = mask ? near_from_slots<TS>(i, n, mask[leaf], near, slots, scale) : near[i];
    double fu = 0.0, fv = 0.0;
    if (has_far) {
        const double cx = x0 + (morton_x(leaf) + 0.5) * w;
        const double cy = y0 + (morton_y(leaf) + 0.5) * w;
        c2<TL> xi;
        if (pos) {
            xi = pos[i];  // the tree's leaf-unit coordinates, made by the same formula
        } else {
            const double2 z = xy[i];
            xi = mk<TL>((TL)((z.x - cx) / w), (TL)((z.y - cy) / w));
        }
        const c2<TL> acc = horner_prefetch<TL>(loc + (int64_t)leaf * p, p, xi);
        fu = (double)acc.x / w;
        fv = -(double)acc.y / w;
    }
    if (staged) {  // at gpos2[i], inside its bucket's window, or else at i
        staged[gpos2 ? gpos2[i] : i] = make_double2(nr.x + fu, nr.y + fv);
        return;
    }
    if (uv) store_velocity(uv, o, make_double2(nr.x + fu, nr.y + fv), base, h);
    if (uv_near) {
        uv_near[2 * o] = nr.x;
        uv_near[2 * o + 1] = nr.y;
    }
    if (uv_far) {
        uv_far[2 * o] = fu;
        uv_far[2 * o + 1] = fv;
    }
}

// Pass 2 of the tree-to-user permutation for large n (the mirror of the circulations'
// two passes): finalize wrote each total at gpos2[i], inside the window of its sorted
// bucket, where the random writes merge in L2; here user row u reads its slot gpos1[u]
// (a chunk of users reads one short run per bucket) and the rows go out in user order.
// The direct scatter to user order (scatter_rows_kernel) makes one random 16-byte write
// per row, which is cheaper while the output is smaller than the chip's 256 MiB last-level
// cache; for 2^25 rows (537 MB) the scatter alone took 1.12 ms, and the windows save 0.3 ms
// per evaluation.  With windows of 2^14 slots (1024 buckets at 2^24 rows) the writes of a
// window stay in the XCD's L2 until their lines are whole: 2^24 patches, 8.35 -> 8.29 ms
// per evaluation against windows of 2^17.
__global__ __launch_bounds__(256) void gather_rows_kernel(int n, int nxcd, const int *__restrict__ gpos1,
                                                          const double2 *__restrict__ staged,
                                                          double *__restrict__ uv, const double *__restrict__ base,
                                                          double h)
{
    const int u = xcd_block(nxcd) * blockDim.x + threadIdx.x;
    if (u >= n) return;
    store_velocity(uv, u, staged[gpos1[u]], base, h);
}

inline unsigned blocks_for(int64_t work, int per_block) { return (unsigned)((work + per_block - 1) / per_block); }

// A grid of whole rounds over the XCDs, for kernels that index blocks with xcd_block.
inline unsigned xcd_grid(int64_t work, int per_block) { return fmm::xcd_grid(work, per_block, kXcds); }


template <typename T> c2<T> *level_ptr(const FarArgs &a, int l, bool local);
template <> double2 *level_ptr<double>(const FarArgs &a, int l, bool local)
{
    return (local ? a.lo_d : a.mp_d) + level_base(l) * a.p;
}
template <> float2 *level_ptr<float>(const FarArgs &a, int l, bool local)
{
    return (local ? a.lo_f : a.mp_f) + (level_base(l) - level_base(a.split + 1)) * a.p;
}

const int *level_list(const fmm_tree *t, int l) { return t->d_lists + t->list_off[l]; }

template <typename TR, typename TC>
void p2m_launch(const FarArgs &a, const FarArgs *b, hipStream_t s)
{
    const fmm_tree *t = a.t;
    const int L = t->depth;
    const int64_t nl = t->list_len[L];
    if (nl == 0) return;
    const double w = t->side / (double)(1 << L);
    c2<TC> *out = level_ptr<TC>(a, L, false);
    // the leaf-unit coordinates when they are in the precision of the expansions
    using TRs = typename RecScalar<TR>::type;
    const c2<TC> *pos = std::is_same<TRs, TC>::value ? (const c2<TC> *)a.pos : nullptr;
    const TRs *gam = (const TRs *)a.gam;
    auto go = [&](auto kernel, int per) {
        kernel<<<dim3(xcd_grid(nl, per), b ? 2 : 1), 64, 0, s>>>(
            level_list(t, L), (int)nl, t->d_leaf_start, t->d_xy, pos, a.gamma.idx, a.gamma.rows, gam, a.adj, t->x0, t->y0, w,
            a.p, out, kXcds, b ? b->adj : nullptr, b ? level_ptr<TC>(*b, L, false) : nullptr);
    };
    // lanes per leaf by the mean occupancy
    const double mean = (double)t->n / (double)nl;
    if (a.p <= 16) {
        if (mean <= 6) go(p2m_kernel<TR, TC, 16, 8>, 8);
        else if (mean <= 32) go(p2m_kernel<TR, TC, 16, 16>, 4);
        else go(p2m_kernel<TR, TC, 16, 32>, 2);
    } else {
        if (mean <= 32) go(p2m_kernel<TR, TC, 32, 16>, 4);
        else go(p2m_kernel<TR, TC, 32, 32>, 2);
    }
}

// ---------------------------------------------------------------------------------
// Backward pass (adjoint of stages 4-10 for a loss L(u)).
// q_i = dL/du_i + i dL/dv_i.  With W = A c and A antisymmetric (A_ij = -A_ji),
//   dL/dGamma_j = -Im((A q)_j)/(2 pi)
// and, with the sources held fixed, dW_i/dx_i = A_i + B_i + W'_far, dW_i/dy_i = i(A_i - B_i + W'_far),
//   A_i = sum_j c_j conj(dz)^2 f'(s),  B_i = sum_j c_j g'(s),   f = g/s, s = |dz|^2,
// so dL/dx_i = Re(q_i (A+B+W')), dL/dy_i = -Im(q_i (A-B+W')).  The particle's own blob
// (dz = 0) contributes B = c_i/(2 sigma^2) and nothing else.
// In the scaled variable s' = alpha^2 |dz|^2 (alpha as in the forward records) and with
// lambda = 1 (FP64, base e) or ln 2 (FP32, base 2):
//   Phi_near = alpha sum_j q_j (g/s') conj(dz'),
//   A = -i alpha^2/(2 pi) sum_j Gamma_j conj(dz')^2 (lambda e s' - g)/s'^2,
//   B = -i alpha^2 lambda/(2 pi) sum_j Gamma_j e,        e = exp(-|dz|^2/(2 sigma^2)), g = 1 - e.
// ---------------------------------------------------------------------------------
// The cotangent reaches tree order as the circulations do: staged by bucket (stage_in_kernel
// on rows of two doubles), then gathered by sorted slot here.
template <typename T>
__global__ __launch_bounds__(256) void pack_adjoint_kernel(int n, int nxcd, const int *__restrict__ gpos2,
                                                            const double2 *__restrict__ dl_st, double scale,
                                                            double2 *__restrict__ adj, c2<T> *__restrict__ qt,
                                                            const double2 *__restrict__ range,
                                                            double *__restrict__ qscale)
{
    const double qs = charge_scale(range, qscale);
    const int i = xcd_block(nxcd) * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const double2 d = dl_st[gpos2[i]];
    const double2 q = make_double2(scale * d.x, scale * d.y);
    adj[i] = q;
    if (qt) qt[i] = mk<T>((T)(qs * q.x), (T)(qs * q.y));
}

// Adjoint near field of one work unit, organised as the forward P2P (LDS tiles,
// exponential skipped on far tiles).  With SRC the source-position sums (At, Bt) go to
// out_src.
template <typename T, bool SRC>
__device__ __forceinline__ void p2p_backward_unit(const int4 u, rec_t<T> *tile, c2<T> *qtile,
                                                  const SoaRec<T> &rec, const c2<T> *__restrict__ qv,
                                                  const int *__restrict__ leaf_start,
                                                  const int *__restrict__ tile_start,
                                                  const float4 *__restrict__ tile_box, int nside, T step,
                                                  float cut_leaf2, float series_leaf2, T lambda,
                                                  double4 *__restrict__ out_pa,
                                                  double4 *__restrict__ out_src)
{
    constexpr int NA = SRC ? 8 : 4;
    const int lane = threadIdx.x;
    const int logtp = u.w;
    const int ix = (int)morton_x((uint32_t)u.x), iy = (int)morton_y((uint32_t)u.x);
    // lane d < 9: the range of neighbour leaf d
    int s0 = 0, slen = 0, ddx = 0, ddy = 0;
    uint32_t SL = 0;
    if (lane < 9) {
        ddx = lane % 3 - 1;
        ddy = lane / 3 - 1;
        const int nx = ix + ddx, ny = iy + ddy;
        if (nx >= 0 && ny >= 0 && nx < nside && ny < nside) {
            SL = morton_encode((uint32_t)nx, (uint32_t)ny);
            s0 = leaf_start[SL];
            slen = leaf_start[SL + 1] - s0;
        }
    }
    if (!__any(slen > 64)) {  // every source leaf is one tile: staged together
        const UnitLanes ul(lane, u.z, logtp);
        const int i = u.y + min(ul.t, u.z - 1);
        const rec_t<T> ri = rec(i);
        bool far = false;
        if (cut_leaf2 < 8.0f && slen > 0) {
            const float4 tbox = tile_box[tile_start[u.x] + ((u.y - leaf_start[u.x]) >> 6)];
            far = box_gap2(tbox, (float)-ddx, (float)-ddy, tile_box[tile_start[SL]]) >= cut_leaf2;
        }
        const T ox = (T)ddx * step, oy = (T)ddy * step;
        double sum[NA] = {};
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
                q = qv[from + j];
            }
            tile[lane] = r;
            qtile[lane] = q;
            r.z = (T)0;
            tile[64 + lane] = r;
            qtile[64 + lane] = mk<T>(0, 0);
        };
        auto fold = [&](const T(&acc)[NA]) {
#pragma unroll
            for (int c = 0; c < NA; ++c) sum[c] += (double)acc[c];
        };
        source_batches<16>(far ? 0 : slen, stage, [&](int count) {
            T acc[NA] = {};
            p2p_bwd_batch<T, false, SRC>(tile, qtile, count, ul.k, ul.K, ri.x, ri.y, lambda, acc);
            fold(acc);
        });
        if (__any(far))
            source_batches<16>(far ? slen : 0, stage, [&](int count) {
                T acc[NA] = {};
                p2p_bwd_batch<T, true, SRC>(tile, qtile, count, ul.k, ul.K, ri.x, ri.y, lambda, acc);
                fold(acc);
            });
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
    const float4 tbox = tile_box[tile_start[u.x] + ((u.y - leaf_start[u.x]) >> 6)];
    double sum[NA] = {};
    for (int dy = -1; dy <= 1; ++dy) {
        const int ny = iy + dy;
        if (ny < 0 || ny >= nside) continue;
        for (int dx = -1; dx <= 1; ++dx) {
            const int nx = ix + dx;
            if (nx < 0 || nx >= nside) continue;
            const uint32_t S = morton_encode((uint32_t)nx, (uint32_t)ny);
            const int s0 = leaf_start[S], s1 = leaf_start[S + 1];
            const T tx = ri.x - (T)dx * step;
            const T ty = ri.y - (T)dy * step;
            T acc[NA] = {};
            int tt = tile_start[S];
            for (int base = s0; base < s1; base += 64, ++tt) {
                const int len = min(64, s1 - base);
                __syncthreads();
                if (lane < len) {
                    tile[lane] = rec(base + lane);
                    qtile[lane] = qv[base + lane];
                }
                const float gap2 = box_gap2(tbox, (float)-dx, (float)-dy, tile_box[tt]);
                const int cls = gap2 >= cut_leaf2 ? 2 : gap2 >= series_leaf2 ? 1 : 0;
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
    }
    for (int o = tp; o < 64; o <<= 1)
#pragma unroll
        for (int c = 0; c < NA; ++c) sum[c] += __shfl_xor(sum[c], o);
    if (k == 0 && t < u.z) {
        out_pa[i] = make_double4(sum[0], sum[1], sum[2], sum[3]);
        if constexpr (SRC) out_src[i] = make_double4(sum[4], sum[5], sum[6], sum[7]);
    }
}

// Adjoint near-field grid: one workgroup per target-centric unit.
template <typename T, bool SRC>
__global__ __launch_bounds__(64, sizeof(T) == 4 ? (SRC ? 5 : 6) : 2) void p2p_backward_kernel(
    const int4 *__restrict__ units, const c2<T> *__restrict__ pos, const T *__restrict__ gam,
    const c2<T> *__restrict__ qv, const int *__restrict__ leaf_start, const int *__restrict__ tile_start,
    const float4 *__restrict__ tile_box, int nside, T step, float cut_leaf2, float series_leaf2, T lambda,
    double4 *__restrict__ out_pa, double4 *__restrict__ out_src)
{
    __shared__ rec_t<T> tile[128];
    __shared__ c2<T> qtile[128];
    const SoaRec<T> rec{pos, gam, step};
    p2p_backward_unit<T, SRC>(units[blockIdx.x], tile, qtile, rec, qv, leaf_start, tile_start, tile_box, nside, step,
                              cut_leaf2, series_leaf2, lambda, out_pa, out_src);
}

// Adjoint finalize: far parts from the q-field locals (Phi_far, by L2P) and the c-field
// locals (W'_far = (1/w^2) sum_l l b_l xi^(l-1)), combined with the near sums.
// Source positions (near_src != NULL): with c = -i Gamma/(2 pi),
//   At = alpha^2 (near sum) + Phi'_far,  Bt = alpha^2 lambda (near sum),
//   dL/dx_src = -Re(c (At + Bt)),  dL/dy_src = Im(c (At - Bt)),
// Phi'_far = (1/w^2) sum_l l b_l(q) xi^(l-1) the derivative of the q-field's local
// expansion (the far operator is antisymmetric).  gamma gives Gamma of sorted
// particle i.
// The far part of a particle's adjoint: Im Phi_far, W'_far and (with need_s) Phi'_far.
struct AdjointFar {
    double phi = 0.0, dwr = 0.0, dwi = 0.0, dpr = 0.0, dpi = 0.0;
};
template <typename TL>
__device__ __forceinline__ AdjointFar adjoint_far(uint32_t leaf, int i, const double2 *__restrict__ xy,
                                                  const c2<TL> *__restrict__ loc_c, const c2<TL> *__restrict__ loc_q,
                                                  const c2<TL> *__restrict__ pos, int p, double x0, double y0,
                                                  double w, bool need_phi, bool need_s)
{
    AdjointFar f;
    c2<TL> xi;
    if (pos) {
        xi = pos[i];
    } else {
        const double cx = x0 + (morton_x(leaf) + 0.5) * w;
        const double cy = y0 + (morton_y(leaf) + 0.5) * w;
        const double2 z = xy[i];
        xi = mk<TL>((TL)((z.x - cx) / w), (TL)((z.y - cy) / w));
    }
    const c2<TL> *bq = loc_q + (int64_t)leaf * p;
    const c2<TL> *bc = loc_c + (int64_t)leaf * p;
    if (need_phi) f.phi = (double)horner_prefetch<TL>(bq, p, xi).y / w;
    if (p >= 2) {
        const c2<TL> accd = horner_weighted_prefetch<TL>(bc, p, xi, 1, 0);
        f.dwr = (double)accd.x / (w * w);
        f.dwi = (double)accd.y / (w * w);
        if (need_s) {
            const c2<TL> accp = horner_weighted_prefetch<TL>(bq, p, xi, 1, 0);
            f.dpr = (double)accp.x / (w * w);
            f.dpi = (double)accp.y / (w * w);
        }
    }
    return f;
}

template <typename TL>
__global__ __launch_bounds__(256) void finalize_backward_kernel(
    int n, const int *__restrict__ perm, const int *__restrict__ leaf_of, const double2 *__restrict__ xy,
    const double4 *__restrict__ near_pa, const double2 *__restrict__ adj,
    const c2<TL> *__restrict__ loc_c, const c2<TL> *__restrict__ loc_q, const c2<TL> *__restrict__ pos, int p,
    int has_far, double x0, double y0,
    double w, double alpha, double lambda, AdjointOut out, const double4 *__restrict__ near_src,
    const int *__restrict__ gpos2, const GammaRows gamma, double *__restrict__ stage_g,
    double *__restrict__ stage_x, double *__restrict__ stage_s, int nxcd)
{
    const bool stage = stage_x != nullptr;
    const bool need_x = out.dxe || out.dxy, need_s = out.dxs || out.dxy;
    const int i = xcd_block(nxcd) * blockDim.x + threadIdx.x;
    if (i >= n) return;
    // the user row, or with stage the staging slot inside the window of the sorted bucket
    const int64_t o = stage ? gpos2[i] : perm[i];  // issued with the first loads
    const double4 a = near_pa[i];
    double phi = alpha * a.x;  // only Im(Phi) enters dL/dGamma
    const double ka = alpha * alpha * kInv2Pi;
    // A = -i ka (a.y + i a.z') with a.z' = -2 a.z (the near sums hold Im A / -2):
    // A = ka (a.z', -a.y);  B = -i ka lambda a.w
    double Ar = ka * (-2.0 * a.z), Ai = -ka * a.y;
    const double Bi = -ka * lambda * a.w;
    double dwr = 0.0, dwi = 0.0, dpr = 0.0, dpi = 0.0;
    if (has_far) {
        const AdjointFar f =
            adjoint_far<TL>((uint32_t)leaf_of[i], i, xy, loc_c, loc_q, pos, p, x0, y0, w, true, need_s);
        phi += f.phi;
        dwr = f.dwr;
        dwi = f.dwi;
        dpr = f.dpr;
        dpi = f.dpi;
    }
    const double g = -phi * kInv2Pi;
    double ex = 0.0, ey = 0.0, sx = 0.0, sy = 0.0;
    if (need_x) {
        const double2 q = adj[i];
        // D1 = A + B + W', D2 = A - B + W'  (B purely imaginary)
        const double d1r = Ar + dwr, d1i = Ai + Bi + dwi;
        const double d2r = Ar + dwr, d2i = Ai - Bi + dwi;
        ex = q.x * d1r - q.y * d1i;
        ey = -(q.x * d2i + q.y * d2r);
    }
    if (need_s) {
        const double4 ns = near_src[i];
        const double a2 = alpha * alpha;
        const double atr = a2 * ns.x + dpr, ati = a2 * ns.y + dpi;
        const double btr = a2 * lambda * ns.z, bti = a2 * lambda * ns.w;
        const double G = gamma.rows[gamma.idx[i]] * kInv2Pi;  // c = -i G: Re(c w) = G Im w, Im(c w) = -G Re w
        sx = -G * (ati + bti);
        sy = -G * (atr - btr);
    }
    if (stage) {  // by staging slot: dL/dGamma, evaluation part, source part
        if (out.dg) stage_g[o] = g;
        if (need_x) {
            stage_x[2 * o] = ex;
            stage_x[2 * o + 1] = ey;
        }
        if (need_s) {
            stage_s[2 * o] = sx;
            stage_s[2 * o + 1] = sy;
        }
        return;
    }
    store_adjoint(out, o, g, ex, ey, sx, sy);
}

// Adjoint finalize of the pair force: the near sums come combined, from the target-centric
// part and the slots as the velocity's; the far parts as above.  (Outputs dl_dxy and dl_dgamma.)
template <typename TL, typename TS>
__global__ __launch_bounds__(256) void finalize_force_kernel(
    int n, const int *__restrict__ perm, const int *__restrict__ leaf_of, const double2 *__restrict__ xy,
    const ForceNear near, const double2 *__restrict__ adj, const c2<TL> *__restrict__ loc_c,
    const c2<TL> *__restrict__ loc_q, const c2<TL> *__restrict__ pos, int p, int has_far, double x0, double y0,
    double w, double alpha, AdjointOut out, const int *__restrict__ gamma_idx, const double *__restrict__ gamma,
    int nxcd)
{
    const int i = xcd_block(nxcd) * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int64_t o = perm[i];  // issued with the first loads
    const uint32_t leaf = (uint32_t)leaf_of[i];
    const double2 q = adj[i];
    const double G = gamma[gamma_idx[i]] * kInv2Pi;
    const int m = near.mask ? near.mask[leaf] : 1 << 9;
    const double uq = near.qscale ? 1.0 / *near.qscale : 1.0;
    const double2 nr = near_from_slots<TS>(i, n, m, near.near, (const c2<TS> *)near.slots, alpha * alpha * kInv2Pi);
    double phi = 0.0;
    if (out.dg) phi = alpha * uq * phi_from_slots<TS>(i, n, m, near.phi, (const TS *)near.phi_slots);
    AdjointFar f;
    if (has_far) f = adjoint_far<TL>(leaf, i, xy, loc_c, loc_q, pos, p, x0, y0, w, out.dg != nullptr, true);
    store_adjoint(out, o, -(phi + f.phi) * kInv2Pi, uq * nr.x + (q.x * f.dwr - q.y * f.dwi),
                  uq * nr.y - (q.x * f.dwi + q.y * f.dwr), -G * f.dpi, -G * f.dpr);
}

// The adjoint outputs from their staging slots (written by finalize_backward_kernel for n
// above the last-level cache) to user order, as gather_rows_kernel does for velocities.
__global__ __launch_bounds__(256) void gather_adjoint_kernel(int n, int nxcd, const int *__restrict__ gpos1,
                                                             const double *__restrict__ stage_g,
                                                             const double *__restrict__ stage_x,
                                                             const double *__restrict__ stage_s, AdjointOut out)
{
    const int u = xcd_block(nxcd) * blockDim.x + threadIdx.x;
    if (u >= n) return;
    const int64_t k = gpos1[u];
    const bool need_x = out.dxe || out.dxy, need_s = out.dxs || out.dxy;
    const double g = out.dg ? stage_g[k] : 0.0;
    const double ex = need_x ? stage_x[2 * k] : 0.0, ey = need_x ? stage_x[2 * k + 1] : 0.0;
    const double sx = need_s ? stage_s[2 * k] : 0.0, sy = need_s ? stage_s[2 * k + 1] : 0.0;
    store_adjoint(out, u, g, ex, ey, sx, sy);
}

// Input check (FMM_OPT_VALIDATE): the lowest particle index whose `stride` values hold a
// NaN or an infinity, by atomic minimum into *first (which starts at INT_MAX).
__global__ void int_fill_kernel(int *p, int v) { *p = v; }

__global__ __launch_bounds__(256) void nonfinite_kernel(int64_t count, int stride, const double *__restrict__ a,
                                                         int *__restrict__ first)
{
    const int64_t step = (int64_t)gridDim.x * blockDim.x;
    for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < count; k += step)
        if (!__builtin_isfinite(a[k])) atomicMin(first, (int)(k / stride));
}

__global__ __launch_bounds__(256) void widen_perm_kernel(int n, const int *__restrict__ perm,
                                                          const int *__restrict__ leaf_of, int64_t *__restrict__ out,
                                                          int32_t *__restrict__ leaf)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    out[i] = perm[i];
    if (leaf) leaf[i] = leaf_of[i];
}

}  // namespace

hipError_t find_nonfinite(const double *a, int64_t n, int stride, int *flag, hipStream_t s, int64_t &bad)
{
    bad = -1;
    const int64_t count = n * stride;
    int_fill_kernel<<<1, 1, 0, s>>>(flag, INT_MAX);
    const unsigned g = (unsigned)std::min<int64_t>(blocks_for(count, 256), 4096);
    nonfinite_kernel<<<g, 256, 0, s>>>(count, stride, a, flag);
    int h = INT_MAX;
    hipError_t e = hipMemcpyAsync(&h, flag, sizeof(int), hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e == hipSuccess && h != INT_MAX) bad = h;
    return e;
}

// ---------------------------------------------------------------------------------
// The static workspace of fmm_velocity_noalloc: per-particle arrays, slots and
// expansions of one call carved from a file-scope device array, for callers that cannot
// allocate.  Host code never uses the array's name as an address: the device address is
// looked up once per device and kept.
// ---------------------------------------------------------------------------------
static __device__ __align__(256) unsigned char scratch[kStaticWorkspaceBytes];

namespace {
__global__ __launch_bounds__(256) void zero_kernel(uint64_t *__restrict__ p, int64_t count)
{
    const int64_t step = (int64_t)gridDim.x * blockDim.x;
    for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < count; k += step) p[k] = 0;
}
}  // namespace

int static_workspace(int device, char **base)
{
    static std::mutex mu;
    static char *ptr[64] = {};
    *base = nullptr;
    if (device < 0 || device >= 64) return (int)hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(mu);
    if (!ptr[device]) {
        void *p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));  // the current device's copy
        if (e != hipSuccess) return (int)e;
        ptr[device] = (char *)p;
    }
    *base = ptr[device];
    return (int)hipSuccess;
}

void launch_zero(void *p, size_t bytes, hipStream_t s)
{
    const int64_t count = (int64_t)(bytes / 8);
    if (count == 0) return;
    zero_kernel<<<(unsigned)std::min<int64_t>(blocks_for(count, 256), 2048), 256, 0, s>>>((uint64_t *)p, count);
}

void launch_widen_perm(const fmm_tree *t, int64_t *perm, int32_t *leaf, hipStream_t s)
{
    const int n = (int)t->n;
    widen_perm_kernel<<<blocks_for(n, 256), 256, 0, s>>>(n, t->d_perm, t->d_leaf_of, perm, leaf);
}

// Grids of the permutation kernels: a multiple of the XCD count (see xcd_block).

void launch_stage_rows(int64_t n, int shift, const int *gpos1, const double *src, double *st, hipStream_t s)
{
    stage_in_kernel<double><<<xcd_grid(n, 256 * kStageE), 256, 0, s>>>((int)n, shift, kXcds, gpos1, src, st);
}

void launch_stage_rows2(int64_t n, int shift, const int *gpos1, const double2 *src, double2 *st, hipStream_t s)
{
    stage_in_kernel<double2><<<xcd_grid(n, 256 * kStageE), 256, 0, s>>>((int)n, shift, kXcds, gpos1, src, st);
}

void launch_gather_rows(int64_t n, const int *gpos1, const double2 *staged, double *uv, const double *base, double h,
                        hipStream_t s)
{
    gather_rows_kernel<<<xcd_grid(n, 256), 256, 0, s>>>((int)n, kXcds, gpos1, staged, uv, base, h);
}

GammaRows launch_stage_in(const fmm_tree *t, const double *gamma, int64_t row, hipStream_t s)
{
    if (direct_rows(t->n, row)) return GammaRows{t->d_perm, gamma};
    launch_stage_rows(t->n, t->stage_shift, t->d_gpos1, gamma, t->d_st1, s);
    return GammaRows{t->d_gpos2, t->d_st1};
}

void launch_pack(const fmm_tree *t, const GammaRows &gamma, int is_double, void *gam, hipStream_t s)
{
    const int n = (int)t->n;
    if (is_double) pack_kernel<double><<<xcd_grid(n, 256), 256, 0, s>>>(n, kXcds, gamma.idx, gamma.rows, (double *)gam);
    else pack_kernel<float><<<xcd_grid(n, 256), 256, 0, s>>>(n, kXcds, gamma.idx, gamma.rows, (float *)gam);
}

void launch_leaf_coords(const fmm_tree *t, int is_double, void *pos, hipStream_t s)
{
    const int n = (int)t->n;
    const double w = t->side / (double)(1 << t->depth);
    if (is_double)
        leaf_coords_kernel<double><<<blocks_for(n, 256), 256, 0, s>>>(n, t->d_leaf_of, t->d_xy, t->x0, t->y0, w,
                                                                      (double2 *)pos);
    else
        leaf_coords_kernel<float><<<blocks_for(n, 256), 256, 0, s>>>(n, t->d_leaf_of, t->d_xy, t->x0, t->y0, w,
                                                                     (float2 *)pos);
}

// Exponential skipped where every pair has s >= cut: FP32 base 2, 1 - 2^-s rounds to 1
// for s >= 26; FP64 base e, 1 - e^-s rounds to 1 for s >= 37.5.  One unit of margin
// covers the rounding of the records and of the box test (boxes in leaf units).
inline float near_cut_leaf2(const fmm_tree *t, int is_double, double alpha)
{
    const double step = alpha * t->side / (double)(1 << t->depth);
    const double cut = is_double ? 39.0 : 27.0;
    return (float)(cut / (step * step));
}

// Dynamic LDS reserved by each near-field workgroup (one wavefront) so that at most
// near_occupancy wavefronts per SIMD are resident (160 KiB of LDS per CU, 4 SIMDs),
// leaving room for the far-field kernels on the other stream.  Serial schedule: no cap.
inline size_t near_lds_reserve(const fmm_tree *t, size_t static_bytes)
{
    if (t->occupancy_in_use <= 0 || t->depth < 2) return 0;
    const size_t per_wave = (size_t)160 * 1024 / (4 * (size_t)t->occupancy_in_use);
    return per_wave > static_bytes ? per_wave - static_bytes : 0;
}

namespace {

MutualParts mutual_parts(const fmm_tree *t, bool mutual)
{
    if (!mutual || t->nsplit == 0) return MutualParts{};
    return MutualParts{t->d_parts, t->d_part_sums, t->npart_sums};
}

template <typename T, int KIND>
void fold_launch(const fmm_tree *t, const MutualParts &parts, void *slots, void *phi, hipStream_t s)
{
    mutual_fold_kernel<T, KIND><<<(unsigned)t->nsplit, 256, 0, s>>>(t->d_split, parts, t->d_leaf_start, t->n,
                                                                    (c2<T> *)slots, (T *)phi);
}

}  // namespace

void launch_p2p_forward(const fmm_tree *t, const void *pos, const void *gam, int is_double, double alpha,
                        double2 *near, void *slots, hipStream_t s)
{
    const bool mutual = slots != nullptr;
    const int64_t nwork = mutual ? t->nnear_work : t->nunits;
    const int4 *work = mutual ? t->d_near_work : t->d_units;
    if (nwork == 0) return;
    const int nside = 1 << t->depth;
    const double w = t->side / (double)nside;
    const double scale = alpha * kInv2Pi;
    const double step = alpha * w;
    const float cut_leaf2 = near_cut_leaf2(t, is_double, alpha);
    const unsigned grid = (unsigned)nwork;
    const MutualParts parts = mutual_parts(t, mutual);
    if (is_double)
        p2p_near_kernel<double><<<grid, 64, near_lds_reserve(t, 256 * sizeof(double4)), s>>>(
            work, (const double2 *)pos, (const double *)gam, t->d_leaf_start, t->d_tile_start,
            t->d_tile_box, nside, step, cut_leaf2, scale, t->dense_leaf, t->n, near, (double2 *)slots, parts);
    else
        p2p_near_kernel<float><<<grid, 64, near_lds_reserve(t, 256 * sizeof(float4)), s>>>(
            work, (const float2 *)pos, (const float *)gam, t->d_leaf_start, t->d_tile_start,
            t->d_tile_box, nside, (float)step, cut_leaf2, scale, t->dense_leaf, t->n, near, (float2 *)slots, parts);
    if (parts.list) {
        if (is_double) fold_launch<double, kVelocity>(t, parts, slots, nullptr, s);
        else fold_launch<float, kVelocity>(t, parts, slots, nullptr, s);
    }
}

namespace {

template <typename T, int KIND>
void force_launch(const fmm_tree *t, const void *pos, const void *gam, const void *qv, const double2 *adj,
                  const GammaRows &gamma, double alpha, const ForceNear &near, hipStream_t s)
{
    const bool mutual = near.slots != nullptr;
    const int64_t nwork = mutual ? t->nnear_work : t->nunits;
    if (nwork == 0) return;
    const int nside = 1 << t->depth;
    const double step = alpha * (t->side / (double)nside);
    const MutualTree mt{t->d_leaf_start, t->d_tile_start, t->d_tile_box, near_cut_leaf2(t, sizeof(T) == 8, alpha),
                        force_series_leaf2(step)};
    const MutualParts parts = mutual_parts(t, mutual);
    p2p_force_kernel<T, KIND><<<(unsigned)nwork, 64, near_lds_reserve(t, sizeof(NearLds<T, KIND>)), s>>>(
        mutual ? t->d_near_work : t->d_units, SoaRec<T>{(const c2<T> *)pos, (const T *)gam, (T)step, (const c2<T> *)qv},
        ForceTargets{adj, gamma, near.qscale}, mt, nside, (T)step, alpha * alpha * kInv2Pi, t->dense_leaf, t->n, near.near, near.phi, (c2<T> *)near.slots,
        (T *)near.phi_slots, parts);
    if (parts.list) fold_launch<T, KIND>(t, parts, near.slots, near.phi_slots, s);
}

}  // namespace

void launch_p2p_force(const fmm_tree *t, const void *pos, const void *gam, const void *qv, const double2 *adj,
                      const GammaRows &gamma, int is_double, double alpha, const ForceNear &near, hipStream_t s)
{
    auto k = is_double ? (near.phi ? force_launch<double, kForcePhi> : force_launch<double, kForce>)
                       : (near.phi ? force_launch<float, kForcePhi> : force_launch<float, kForce>);
    k(t, pos, gam, qv, adj, gamma, alpha, near, s);
}

namespace {

void launch_p2m(const FarArgs &a, const FarArgs *b, hipStream_t s)
{
    auto k = a.t->depth <= a.split ? (a.rec_is_double ? p2m_launch<double4, double> : p2m_launch<float4, double>)
                                   : (a.rec_is_double ? p2m_launch<double4, float> : p2m_launch<float4, float>);
    k(a, b, s);
}

// The target segments of levels l0..l1 for one launch: the four parity classes of each.
void class_segs(TransArgs &a, const fmm_tree *t, int l0, int l1)
{
    a.nseg = 0;
    for (int l = l0; l <= l1; ++l)
        for (int q = 0; q < 4; ++q) {
            const int64_t *co = &t->class_off[4 * l];
            TransSeg &g = a.seg[a.nseg++];
            g.start = (int)(t->list_off[l] + co[q]);
            g.len = (int)((q < 3 ? co[q + 1] : t->list_len[l]) - co[q]);
            g.level = l;
        }
}

}  // namespace

// Stage 5 up to level 2, stage 6 (M2L) for every level but the widest at once (one launch
// per precision), stage 7 down, with the M2L of the widest levels.  FP64 levels that a 1024-workgroup grid covers run three to a launch
// (launch_subtree); the rest one level to a launch.
void launch_far_chain(const FarArgs &a, hipStream_t s, const FarArgs *b)
{
    const fmm_tree *t = a.t;
    const int L = t->depth;
    if (L < 2) return;
    const Tables &tb = *t->tabs;
    launch_p2m(a, b, s);  // stage 4
    const int S = std::min(L, a.split);  // last FP64 level
    const int64_t fbase = level_base(a.split + 1);

    TransArgs g{};
    g.p = a.p;
    g.no_lds = a.no_lds;
    g.targets = t->d_lists;
    g.entries = tb.mfma_entries;
    g.zero = tb.zero_row;
    SubtreeArgs st{};
    st.p = a.p;
    st.deepest = S;
    st.counts = t->d_counts;
    st.tab = tb.mfma_d;

    // the source and target rows of both sets
    auto set = [&](TransArgs &to, auto rows) {
        rows(a, to.src, to.out);
        if (b) rows(*b, to.src2, to.out2);
    };
    // the group of three levels a subtree launch covers: bases 2 and 5 (16 and 1024 workgroups)
    auto group = [](int rank) { return 2 + 3 * (rank / 3); };

    for (int l = L - 1; l >= 2;) {
        g.nseg = 1;
        g.seg[0] = TransSeg{0, (int)t->list_off[l], (int)t->list_len[l], l};
        if (l >= a.split) {  // FP32 children
            g.tab = tb.mfma_f;
            set(g, [&](const FarArgs &f, const void *&src, void *&out) {
                src = f.mp_f;
                out = l == f.split ? (void *)f.mp_d : (void *)f.mp_f;
            });
            g.src_off = fbase;
            g.out_off = l == a.split ? 0 : fbase;
            launch_trans32(g, Trans::M2M, false, l == a.split, s);
            --l;
            continue;
        }
        const int base = group(l - 2);
        if (base == 2 || (base == 5 && l > 5)) {
            st.base = base;
            st.rows = (double *)a.mp_d;
            st.rows2 = b ? (double *)b->mp_d : nullptr;
            st.deepest = l + 1;
            launch_subtree(st, true, s);
            l = base - 1;
            continue;
        }
        g.tab = tb.mfma_d;
        set(g, [](const FarArgs &f, const void *&src, void *&out) { src = out = f.mp_d; });
        g.src_off = g.out_off = 0;
        launch_trans64(g, Trans::M2M, false, s);
        --l;
    }

    // levels from wide on (the finest, where the tree has cells enough) take M2L and L2L together
    int wide = L + 1;
    while (wide > 3 && wide - 1 != S + 1 &&  // (the parents in the level's own precision)
           (wide - 1 > S ? wide_level32(t->list_len[wide - 1], a.p) : wide_level64(t->list_len[wide - 1], a.p)))
        --wide;
    class_segs(g, t, 2, std::min(S, wide - 1));
    g.tab = tb.mfma_d;
    set(g, [](const FarArgs &f, const void *&src, void *&out) {
        src = f.mp_d;
        out = f.lo_d;
    });
    g.src_off = g.out_off = 0;
    launch_trans64(g, Trans::M2L, false, s);
    if (wide - 1 > S) {
        class_segs(g, t, S + 1, wide - 1);
        g.tab = tb.mfma_f;
        set(g, [](const FarArgs &f, const void *&src, void *&out) {
            src = f.mp_f;
            out = f.lo_f;
        });
        g.src_off = g.out_off = fbase;
        launch_trans32(g, Trans::M2L, false, false, s);
    }

    for (int l = 3; l <= L;) {
        if (l >= wide) {
            class_segs(g, t, l, l);
            set(g, [&](const FarArgs &f, const void *&src, void *&out) {
                src = l <= S ? (const void *)f.mp_d : (const void *)f.mp_f;
                out = l <= S ? (void *)f.lo_d : (void *)f.lo_f;
            });
            g.par = g.out;
            g.par2 = g.out2;
            g.par_off = l <= S ? 0 : fbase;
            g.tab = l <= S ? (const void *)tb.mfma_d : (const void *)tb.mfma_f;
            g.src_off = g.out_off = l <= S ? 0 : fbase;
            if (l <= S) launch_trans64(g, Trans::M2L, false, s);
            else launch_trans32(g, Trans::M2L, false, false, s);
            g.par = g.par2 = nullptr;
            ++l;
            continue;
        }
        if (l > S) {  // FP32 targets
            class_segs(g, t, l, l);
            g.tab = tb.mfma_f;
            set(g, [&](const FarArgs &f, const void *&src, void *&out) {
                src = l - 1 <= S ? (const void *)f.lo_d : (const void *)f.lo_f;
                out = f.lo_f;
            });
            g.src_off = l - 1 <= S ? 0 : fbase;
            g.out_off = fbase;
            launch_trans32(g, Trans::L2L, l - 1 <= S, false, s);
            ++l;
            continue;
        }
        const int base = group(l - 3), last = std::min({S, base + 3, wide - 1});
        if (base == 2 || (base == 5 && last > 6)) {
            st.base = base;
            st.rows = (double *)a.lo_d;
            st.rows2 = b ? (double *)b->lo_d : nullptr;
            st.deepest = last;
            launch_subtree(st, false, s);
            l = last + 1;
            continue;
        }
        class_segs(g, t, l, l);
        g.tab = tb.mfma_d;
        set(g, [](const FarArgs &f, const void *&src, void *&out) { src = out = f.lo_d; });
        g.src_off = g.out_off = 0;
        launch_trans64(g, Trans::L2L, false, s);
        ++l;
    }
}

void launch_finalize(const fmm_tree *t, const FarArgs &a, const double2 *near, const void *slots, int slots_double,
                     double alpha, double *uv, double *uv_near, double *uv_far, void *stage, const double *base,
                     double h, hipStream_t s)
{
    // uv alone: the totals go to stage (n double2), then out in user order; through the
    // staging windows once the output outgrows the last-level cache; small outputs directly
    double2 *staged = uv && !uv_near && !uv_far && !direct_rows(t->n, kForwardRow) ? (double2 *)stage : nullptr;
    const bool windowed = outputs_windowed(t->n, sizeof(double2));
    double *uv_direct = staged ? nullptr : uv;
    const int L = t->depth;
    const int n = (int)t->n;
    const double w = t->side / (double)(1 << L);
    const int has_far = L >= 2;
    const uint16_t *mask = slots ? t->d_leaf_mask : nullptr;
    const double scale = alpha * kInv2Pi;
    const dim3 g(xcd_grid(n, 256));
    const int *gp = windowed ? t->d_gpos2 : nullptr;
    // L2P at the tree's leaf-unit coordinates when they are in the precision of the locals
    if (!has_far || L <= a.split) {
        const double2 *loc = has_far ? level_ptr<double>(a, L, true) : nullptr;
        const double2 *pos = a.rec_is_double ? (const double2 *)a.pos : nullptr;
        if (slots_double)
            finalize_kernel<double, double><<<g, 256, 0, s>>>(n, t->d_perm, t->d_leaf_of, t->d_xy, near, mask,
                                                              (const double2 *)slots, scale, loc, pos, a.p, has_far,
                                                              t->x0, t->y0, w, uv_direct, uv_near, uv_far, staged, gp,
                                                              kXcds, base, h);
        else
            finalize_kernel<double, float><<<g, 256, 0, s>>>(n, t->d_perm, t->d_leaf_of, t->d_xy, near, mask,
                                                             (const float2 *)slots, scale, loc, pos, a.p, has_far,
                                                             t->x0, t->y0, w, uv_direct, uv_near, uv_far, staged, gp,
                                                             kXcds, base, h);
    } else {
        const float2 *loc = level_ptr<float>(a, L, true);
        const float2 *pos = a.rec_is_double ? nullptr : (const float2 *)a.pos;
        if (slots_double)
            finalize_kernel<float, double><<<g, 256, 0, s>>>(n, t->d_perm, t->d_leaf_of, t->d_xy, near, mask,
                                                             (const double2 *)slots, scale, loc, pos, a.p, has_far,
                                                             t->x0, t->y0, w, uv_direct, uv_near, uv_far, staged, gp,
                                                             kXcds, base, h);
        else
            finalize_kernel<float, float><<<g, 256, 0, s>>>(n, t->d_perm, t->d_leaf_of, t->d_xy, near, mask,
                                                            (const float2 *)slots, scale, loc, pos, a.p, has_far,
                                                            t->x0, t->y0, w, uv_direct, uv_near, uv_far, staged, gp,
                                                            kXcds, base, h);
    }
    if (staged && windowed) gather_rows_kernel<<<g, 256, 0, s>>>(n, kXcds, t->d_gpos1, staged, uv, base, h);
    else if (staged) scatter_rows_kernel<<<blocks_for(n, 256), 256, 0, s>>>(n, t->d_perm, staged, uv, base, h);
}
void launch_adjoint_range(int64_t n, const double *gamma, const double *dl_duv, double scale, double2 *range,
                          hipStream_t s)
{
    adjoint_range_kernel<<<kRangeBlocks, 256, 0, s>>>(n, gamma, (const double2 *)dl_duv, scale, range);
}

void launch_pack_adjoint(const fmm_tree *t, const double *dl_duv, double scale, double2 *adj, void *qt, int is_double,
                         double2 *staging, const double2 *range, double *qscale, hipStream_t s)
{
    const int n = (int)t->n;
    const bool direct = direct_rows(n, kAdjointRow);
    const int *idx = direct ? t->d_perm : t->d_gpos2;
    const double2 *rows = direct ? (const double2 *)dl_duv : staging;
    if (!direct) launch_stage_rows2(n, t->stage_shift, t->d_gpos1, (const double2 *)dl_duv, staging, s);
    if (is_double)
        pack_adjoint_kernel<double><<<xcd_grid(n, 256), 256, 0, s>>>(n, kXcds, idx, rows, scale, adj,
                                                                      nullptr, nullptr, nullptr);
    else
        pack_adjoint_kernel<float><<<xcd_grid(n, 256), 256, 0, s>>>(n, kXcds, idx, rows, scale, adj,
                                                                     (float2 *)qt, range, qscale);
}

void launch_p2p_backward(const fmm_tree *t, const void *pos, const void *gam, const void *qv, int is_double,
                         double alpha,
                         double4 *out_pa, double4 *out_src, hipStream_t s)
{
    if (t->nunits == 0) return;
    const int nside = 1 << t->depth;
    const double w = t->side / (double)nside;
    const double step = alpha * w;
    const double cut = is_double ? 39.0 : 27.0;
    const float cut_leaf2 = (float)(cut / (step * step));
    const unsigned grid = (unsigned)t->nunits;
    const double ln2 = 0.69314718055994530942;
    // the series of the pair code applies below s' = (0.125 / ln 2) in FP32 (natural exponent
    // 0.125) and 1e-3 in FP64; tiles whose boxes are twice that apart skip the test
    const double series_s = is_double ? 1e-3 : 0.125 / ln2;
    const float series_leaf2 = (float)(2.0 * series_s / (step * step));
    if (is_double) {
        if (out_src)
            p2p_backward_kernel<double, true><<<grid, 64, 0, s>>>(
                t->d_units, (const double2 *)pos, (const double *)gam, (const double2 *)qv, t->d_leaf_start,
                t->d_tile_start, t->d_tile_box, nside, step, cut_leaf2, series_leaf2, 1.0, out_pa, out_src);
        else
            p2p_backward_kernel<double, false><<<grid, 64, 0, s>>>(
                t->d_units, (const double2 *)pos, (const double *)gam, (const double2 *)qv, t->d_leaf_start,
                t->d_tile_start, t->d_tile_box, nside, step, cut_leaf2, series_leaf2, 1.0, out_pa, nullptr);
    } else {
        if (out_src)
            p2p_backward_kernel<float, true><<<grid, 64, 0, s>>>(
                t->d_units, (const float2 *)pos, (const float *)gam, (const float2 *)qv, t->d_leaf_start,
                t->d_tile_start, t->d_tile_box, nside, (float)step, cut_leaf2, series_leaf2, (float)ln2, out_pa,
                out_src);
        else
            p2p_backward_kernel<float, false><<<grid, 64, 0, s>>>(
                t->d_units, (const float2 *)pos, (const float *)gam, (const float2 *)qv, t->d_leaf_start,
                t->d_tile_start, t->d_tile_box, nside, (float)step, cut_leaf2, series_leaf2, (float)ln2, out_pa,
                nullptr);
    }
}

namespace {

template <typename TL, typename TS>
void finalize_force_launch(const fmm_tree *t, const FarArgs &fc, const FarArgs &fq, const double2 *adj,
                           const ForceNear &near, double alpha, const AdjointOut &out, hipStream_t s)
{
    const int L = t->depth;
    const bool has_far = L >= 2;
    finalize_force_kernel<TL, TS><<<xcd_grid(t->n, 256), 256, 0, s>>>(
        (int)t->n, t->d_perm, t->d_leaf_of, t->d_xy, near, adj, has_far ? level_ptr<TL>(fc, L, true) : nullptr,
        has_far ? level_ptr<TL>(fq, L, true) : nullptr,
        (fc.rec_is_double != 0) == (sizeof(TL) == 8) ? (const c2<TL> *)fc.pos : nullptr, fc.p, has_far, t->x0, t->y0,
        t->side / (double)(1 << L), alpha, out, fc.gamma.idx, fc.gamma.rows, kXcds);
}

}  // namespace

void launch_finalize_force(const fmm_tree *t, const FarArgs &fc, const FarArgs &fq, const double2 *adj,
                           const ForceNear &near, int is_double, double alpha, const AdjointOut &out, hipStream_t s)
{
    auto k = t->depth < 2 || t->depth <= fc.split
                 ? (is_double ? finalize_force_launch<double, double> : finalize_force_launch<double, float>)
                 : (is_double ? finalize_force_launch<float, double> : finalize_force_launch<float, float>);
    k(t, fc, fq, adj, near, alpha, out, s);
}

void launch_finalize_backward(const fmm_tree *t, const FarArgs &fc, const FarArgs &fq, const double4 *near_pa,
                              const double2 *adj, const double4 *near_src, int is_double,
                              double alpha, const AdjointOut &out, double *stage_g, double *stage_x,
                              double *stage_s, hipStream_t s)
{
    const int L = t->depth;
    const int n = (int)t->n;
    const dim3 g(xcd_grid(n, 256));
    const double w = t->side / (double)(1 << L);
    const int has_far = L >= 2;
    const double lambda = is_double ? 1.0 : 0.69314718055994530942;
    if (!has_far || L <= fc.split)
        finalize_backward_kernel<double><<<g, 256, 0, s>>>(
            n, t->d_perm, t->d_leaf_of, t->d_xy, near_pa, adj,
            has_far ? level_ptr<double>(fc, L, true) : nullptr, has_far ? level_ptr<double>(fq, L, true) : nullptr,
            fc.rec_is_double ? (const double2 *)fc.pos : nullptr, fc.p, has_far, t->x0, t->y0, w, alpha, lambda, out, near_src, t->d_gpos2, fc.gamma, stage_g, stage_x,
            stage_s, kXcds);
    else
        finalize_backward_kernel<float><<<g, 256, 0, s>>>(
            n, t->d_perm, t->d_leaf_of, t->d_xy, near_pa, adj, level_ptr<float>(fc, L, true),
            level_ptr<float>(fq, L, true), fc.rec_is_double ? nullptr : (const float2 *)fc.pos, fc.p, has_far, t->x0, t->y0, w, alpha, lambda, out, near_src, t->d_gpos2,
            fc.gamma, stage_g, stage_x, stage_s, kXcds);
    if (stage_x) gather_adjoint_kernel<<<g, 256, 0, s>>>(n, kXcds, t->d_gpos1, stage_g, stage_x, stage_s, out);
}


}  // namespace fmm
