// Stages 1-3 of Fig. fmmStages on the GPU: root cell, binning, Morton sort, leaf
// offsets, per-level occupancy, interaction-list cell lists, near-field work lists and
// the statistics of fmm_tree_info.
//
// The arrays equal those of the host build (host_tree.cpp) element for element (same
// arithmetic for the binning and tile boxes, stable sorts with the same keys, the cost
// orders included), so either build gives bit-identical evaluations.  The building blocks are a stable LSD radix
// sort of (64-bit key, 32-bit value) pairs with 8-bit digits and a device-wide
// exclusive scan, both written here.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <vector>

#include "../../include/fmm2d.h"
#include "build_prims.h"
#include "fmm_internal.h"

namespace fmm {

namespace {

// ---------------------------------------------------------------------------------
// Device-wide exclusive scan of uint32 (totals below 2^32).  Tiles of 2048: each
// thread scans 8 consecutive elements, the block scans the thread totals; the tile sums
// before a tile are added up by its workgroup.  In place is allowed.
// ---------------------------------------------------------------------------------
constexpr int kScanTile = 2048;

__device__ inline uint32_t block_exclusive_sum(uint32_t v, uint32_t &total)
{
    __shared__ uint32_t wsum[4];
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    uint32_t x = v;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t y = __shfl_up(x, d);
        if (lane >= d) x += y;
    }
    if (lane == 63) wsum[wid] = x;
    __syncthreads();
    uint32_t before = 0;
    total = 0;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        if (w < wid) before += wsum[w];
        total += wsum[w];
    }
    __syncthreads();
    return before + x - v;
}

__global__ __launch_bounds__(256) void scan_tile_sums(const uint32_t *__restrict__ in, int64_t n,
                                                       uint32_t *__restrict__ sums)
{
    const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * 8;
    uint32_t s = 0;
#pragma unroll
    for (int e = 0; e < 8; ++e)
        if (base + e < n) s += in[base + e];
    uint32_t total;
    block_exclusive_sum(s, total);
    if (threadIdx.x == 0) sums[blockIdx.x] = total;
}

// Each workgroup adds up the sums of the tiles before its own (at most kScanSelf of them,
// so reading them costs less than a launch of its own for their scan).
constexpr int kScanSelf = 8192;

__global__ __launch_bounds__(256) void scan_tiles(const uint32_t *in, uint32_t *out, int64_t n,
                                                   const uint32_t *__restrict__ sums, uint32_t *__restrict__ total)
{
    uint32_t before = 0, part = 0;
    for (int k = threadIdx.x; k < (int)blockIdx.x; k += 256) part += sums[k];
    block_exclusive_sum(part, before);
    const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * 8;
    uint32_t v[8], s = 0;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        v[e] = base + e < n ? in[base + e] : 0u;
        s += v[e];
    }
    uint32_t tot;
    uint32_t run = before + block_exclusive_sum(s, tot);
#pragma unroll
    for (int e = 0; e < 8; ++e)
        if (base + e < n) {
            out[base + e] = run;
            run += v[e];
        }
    if (total && blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) *total = before + tot;
}

// As scan_tiles with the exclusive sums before each tile already made.
__global__ __launch_bounds__(256) void scan_add(const uint32_t *in, uint32_t *out, int64_t n,
                                                 const uint32_t *__restrict__ sums, uint32_t *__restrict__ total)
{
    const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * 8;
    uint32_t v[8], s = 0;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        v[e] = base + e < n ? in[base + e] : 0u;
        s += v[e];
    }
    uint32_t tot;
    uint32_t run = sums[blockIdx.x] + block_exclusive_sum(s, tot);
#pragma unroll
    for (int e = 0; e < 8; ++e)
        if (base + e < n) {
            out[base + e] = run;
            run += v[e];
        }
    if (total && blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) *total = sums[blockIdx.x] + tot;
}

// Short arrays in one workgroup, tile after tile.
__global__ __launch_bounds__(256) void scan_short(const uint32_t *in, uint32_t *out, int64_t n,
                                                   uint32_t *__restrict__ total)
{
    uint32_t carry = 0;
    for (int64_t t0 = 0; t0 < n; t0 += kScanTile) {
        const int64_t base = t0 + (int64_t)threadIdx.x * 8;
        uint32_t v[8], s = 0;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            v[e] = base + e < n ? in[base + e] : 0u;
            s += v[e];
        }
        uint32_t tot;
        uint32_t run = carry + block_exclusive_sum(s, tot);
#pragma unroll
        for (int e = 0; e < 8; ++e)
            if (base + e < n) {
                out[base + e] = run;
                run += v[e];
            }
        carry += tot;
    }
    if (total && threadIdx.x == 0) *total = carry;
}

// ---------------------------------------------------------------------------------
// Stable LSD radix sort of (key, value) pairs by the low `bits` bits of the key,
// 8-bit digits.  Per pass: per-tile digit histograms (digit-major), their exclusive scan within
// each digit, then a scatter in which each tile of 256 R pairs is taken in R rounds of 256;
// inside a wavefront the lanes with the same digit find each other with 8 ballots
// (rank = lanes below with the same digit), across wavefronts and rounds the digit
// counts accumulate in LDS, so equal digits keep their input order.  Small sorts are a chain of
// launches and round trips to memory: the scatter adds up the digits' totals itself instead of a
// scan over all counts (of 1000003 pairs: 8 us and two launches a pass, now 3.3 and one), a tile's
// pairs are all loaded before its first round, and up to kSmallSort pairs a tile is two rounds
// (scatter of 12289 pairs 8.2 -> 3.8 us; of 1000003 pairs 14.8 us with eight rounds, 16.2 with
// four, 13.6 with two, whose counts then cost more: 2.10, 2.13 and 2.22 ms of an RK2 step).
// ---------------------------------------------------------------------------------
constexpr int64_t kSmallSort = int64_t(1) << 18;  // pairs up to which a tile is two rounds

template <int R>
__global__ __launch_bounds__(256) void rs_hist(const uint64_t *__restrict__ keys, int64_t n, int shift,
                                                uint32_t *__restrict__ counts, int nb)
{
    __shared__ uint32_t h[256];
    h[threadIdx.x] = 0;
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * (256 * R) + threadIdx.x;
    uint32_t d[R];
#pragma unroll
    for (int r = 0; r < R; ++r) d[r] = base + r * 256 < n ? (uint32_t)(keys[base + r * 256] >> shift) & 255u : 256u;
#pragma unroll
    for (int r = 0; r < R; ++r)
        if (d[r] < 256u) atomicAdd(&h[d[r]], 1u);
    __syncthreads();
    counts[(int64_t)threadIdx.x * nb + blockIdx.x] = h[threadIdx.x];
}

// Exclusive sum over a workgroup of 256 threads, and the total.
__device__ __forceinline__ uint32_t block_scan(uint32_t v, uint32_t &total)
{
    __shared__ uint32_t wsum[4];
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    uint32_t incl = v;
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t u = __shfl_up(incl, o);
        if (lane >= o) incl += u;
    }
    __syncthreads();  // (a caller's earlier sum)
    if (lane == 63) wsum[wid] = incl;
    __syncthreads();
    uint32_t before = 0;
    for (int w = 0; w < 4; ++w) before += w < wid ? wsum[w] : 0u;
    total = wsum[0] + wsum[1] + wsum[2] + wsum[3];
    return before + incl - v;
}

// Per digit (workgroup): its tiles' counts to exclusive offsets within the digit, and its total.
__global__ __launch_bounds__(256) void rs_scan(uint32_t *__restrict__ counts, int nb, uint32_t *__restrict__ totals)
{
    uint32_t *c = counts + (int64_t)blockIdx.x * nb;
    uint32_t carry = 0;
    for (int b = 0; b < nb; b += 256) {
        const int k = b + threadIdx.x;
        uint32_t total;
        const uint32_t e = block_scan(k < nb ? c[k] : 0u, total);
        if (k < nb) c[k] = carry + e;
        carry += total;
    }
    if (threadIdx.x == 0) totals[blockIdx.x] = carry;
}

template <int R>
__global__ __launch_bounds__(256) void rs_scatter(const uint64_t *__restrict__ kin, const uint32_t *__restrict__ vin,
                                                   uint64_t *__restrict__ kout, uint32_t *__restrict__ vout, int64_t n,
                                                   int shift, const uint32_t *__restrict__ offs, int nb,
                                                   const uint32_t *__restrict__ totals)
{
    __shared__ uint32_t start[256];
    __shared__ uint32_t wcnt[4][256];
    const int t = threadIdx.x, lane = t & 63, wid = t >> 6;
    const int64_t base = (int64_t)blockIdx.x * (256 * R) + t;
    uint64_t key[R];
    uint32_t val[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int64_t i = min(base + r * 256, n - 1);
        key[r] = kin[i];
        val[r] = vin[i];
    }
    uint32_t all;
    start[t] = offs[(int64_t)t * nb + blockIdx.x] + block_scan(totals[t], all);
#pragma unroll
    for (int r = 0; r < R; ++r) {
        wcnt[0][t] = wcnt[1][t] = wcnt[2][t] = wcnt[3][t] = 0;
        __syncthreads();
        const bool valid = base + r * 256 < n;
        const uint32_t d = (uint32_t)(key[r] >> shift) & 255u;
        uint64_t m = __ballot(valid);
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            const bool bit = (d >> b) & 1u;
            const uint64_t bm = __ballot(valid && bit);
            m &= bit ? bm : ~bm;
        }
        const uint64_t below = m & ((1ull << lane) - 1ull);
        if (valid && below == 0) wcnt[wid][d] = (uint32_t)__popcll(m);  // lowest lane of its digit group
        __syncthreads();
        if (valid) {
            uint32_t pos = start[d] + (uint32_t)__popcll(below);
            for (int w = 0; w < wid; ++w) pos += wcnt[w][d];
            kout[pos] = key[r];
            vout[pos] = val[r];
        }
        __syncthreads();
        start[t] += wcnt[0][t] + wcnt[1][t] + wcnt[2][t] + wcnt[3][t];
    }
}

// All passes of a small sort in one workgroup of 16 wavefronts: a pass above costs three launches
// of 3 us each.  A wavefront takes 64 consecutive pairs a round, in order, and counts its digits
// apart, so that its rounds need no barrier: the places of its digits (after those of lower digits
// and of earlier wavefronts) advance as it goes.  One compute unit does the work of all, so the
// line lies where its rounds take as long as the launches: a stage with its rebuild of 4097
// uniform particles 326 -> 292 us, 8001 328 -> 307; up to 16384 pairs 12289 particles take 321
// instead of 307, 16001 take 336 instead of 312 (325 before).
constexpr int64_t kOneSort = 8192;

template <int R>
__global__ __launch_bounds__(1024) void rs_one(uint64_t *ka, uint32_t *va, uint64_t *kb, uint32_t *vb, int n, int bits)
{
    __shared__ uint32_t place[16][256];
    __shared__ uint32_t wsum[4];
    const int t = threadIdx.x, lane = t & 63, wid = t >> 6;
    const int rounds = (n + 1023) / 1024;  // at most R
    const int first = wid * 64 * rounds + lane;
    for (int shift = 0; shift < bits; shift += 8) {
        uint64_t key[R];
        uint32_t val[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int i = min(first + r * 64, n - 1);
            key[r] = ka[i];
            val[r] = va[i];
        }
        for (int k = 0; k < 4; ++k) (&place[0][0])[k * 1024 + t] = 0;
        __syncthreads();
#pragma unroll
        for (int r = 0; r < R; ++r)
            if (r < rounds && first + r * 64 < n) atomicAdd(&place[wid][(key[r] >> shift) & 255u], 1u);
        __syncthreads();
        uint32_t total = 0, incl = 0;
        if (t < 256) {  // digit t
            for (int w = 0; w < 16; ++w) {
                const uint32_t c = place[w][t];
                place[w][t] = total;
                total += c;
            }
            incl = total;
            for (int o = 1; o < 64; o <<= 1) {
                const uint32_t u = __shfl_up(incl, o);
                if (lane >= o) incl += u;
            }
            if (lane == 63) wsum[wid] = incl;
        }
        __syncthreads();
        if (t < 256) {
            uint32_t before = incl - total;
            for (int w = 0; w < wid; ++w) before += wsum[w];
            for (int w = 0; w < 16; ++w) place[w][t] += before;
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if (r >= rounds) break;
            const bool valid = first + r * 64 < n;
            const uint32_t d = (uint32_t)(key[r] >> shift) & 255u;
            uint64_t m = __ballot(valid);
#pragma unroll
            for (int b = 0; b < 8; ++b) {
                const bool bit = (d >> b) & 1u;
                const uint64_t bm = __ballot(valid && bit);
                m &= bit ? bm : ~bm;
            }
            const uint64_t below = m & ((1ull << lane) - 1ull);
            const uint32_t at = place[wid][d];
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            if (valid && below == 0) place[wid][d] = at + (uint32_t)__popcll(m);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            if (valid) {
                const uint32_t pos = at + (uint32_t)__popcll(below);
                kb[pos] = key[r];
                vb[pos] = val[r];
            }
        }
        __syncthreads();
        uint64_t *const k = ka;
        ka = kb;
        kb = k;
        uint32_t *const v = va;
        va = vb;
        vb = v;
    }
}

// ---------------------------------------------------------------------------------
// Tree kernels
// ---------------------------------------------------------------------------------
// What a uniform build reports to the host, read back twice: after the keys (the checks
// and the root cell) and after the counts (the sizes of the lists).
// target-centric units, mutual items, mutual pairs, estimated cost; split items, their parts and
// the places in the parts' sums; then how many of these three are given out
enum PlanFact { kPlanUnits, kPlanItems, kPlanPairs, kPlanCost, kPlanSplit, kPlanParts, kPlanSums, kPlanNext, kPlanFacts = 10 };
struct BuildFacts {
    int flags;                    // k_minmax, k_keys
    unsigned long long first_bad;
    double x0, y0, side;
    uint32_t ntiles, nlist, nwork;
    uint32_t class_off[4 * (kMaxDepth + 1)];
    unsigned long long plan[kPlanFacts];  // see PlanFact
    unsigned long long stats[4];  // near pairs (with the particle itself), non-empty leaves, largest, M2L pairs
};

__global__ void k_facts(BuildFacts *f, double x0, double y0, double side)
{
    *f = BuildFacts{};
    f->first_bad = ~0ull;
    f->x0 = x0;
    f->y0 = y0;
    f->side = side;
}

// Per-block min/max of the coordinates; flags bit 2: a non-finite coordinate.
__global__ __launch_bounds__(256) void k_minmax(const double2 *__restrict__ xy, int64_t n, double4 *__restrict__ part,
                                                 int *__restrict__ flags, int nonfinite_bit)
{
    double xmin = INFINITY, xmax = -INFINITY, ymin = INFINITY, ymax = -INFINITY;
    bool bad = false;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const double2 z = xy[i];
        if (!isfinite(z.x) || !isfinite(z.y)) {
            bad = true;
            continue;
        }
        xmin = fmin(xmin, z.x);
        xmax = fmax(xmax, z.x);
        ymin = fmin(ymin, z.y);
        ymax = fmax(ymax, z.y);
    }
    if (bad) atomicOr(flags, nonfinite_bit);
    for (int o = 32; o > 0; o >>= 1) {
        xmin = fmin(xmin, __shfl_xor(xmin, o));
        xmax = fmax(xmax, __shfl_xor(xmax, o));
        ymin = fmin(ymin, __shfl_xor(ymin, o));
        ymax = fmax(ymax, __shfl_xor(ymax, o));
    }
    __shared__ double4 w[4];
    if ((threadIdx.x & 63) == 0) w[threadIdx.x >> 6] = make_double4(xmin, xmax, ymin, ymax);
    __syncthreads();
    if (threadIdx.x == 0) {
        double4 r = w[0];
        for (int k = 1; k < 4; ++k) {
            r.x = fmin(r.x, w[k].x);
            r.y = fmax(r.y, w[k].y);
            r.z = fmin(r.z, w[k].z);
            r.w = fmax(r.w, w[k].w);
        }
        part[blockIdx.x] = r;
    }
}

// The bounding square from the block results: {x0, y0, side} = (min x, min y, largest range
// (1 + 2^-20)), side 1 for a single point.
__global__ __launch_bounds__(256) void k_root(const double4 *__restrict__ part, int nb, BuildFacts *__restrict__ f)
{
    __shared__ double4 w[256];
    double4 r = part[min((int)threadIdx.x, nb - 1)];
    for (int k = threadIdx.x + 256; k < nb; k += 256) {
        r.x = fmin(r.x, part[k].x);
        r.y = fmax(r.y, part[k].y);
        r.z = fmin(r.z, part[k].z);
        r.w = fmax(r.w, part[k].w);
    }
    w[threadIdx.x] = r;
    __syncthreads();
    if (threadIdx.x) return;
    for (int k = 1; k < 256; ++k) {
        r.x = fmin(r.x, w[k].x);
        r.y = fmax(r.y, w[k].y);
        r.z = fmin(r.z, w[k].z);
        r.w = fmax(r.w, w[k].w);
    }
    double side = fmax(r.y - r.x, r.w - r.z);
    if (!(side > 0.0)) side = 1.0;
    f->x0 = r.x;
    f->y0 = r.z;
    f->side = side * (1.0 + 1.0 / 1048576.0);
}

// Leaf (floor binning, clamped at the top edge) and sub-leaf key (64 x 64 grid over the
// leaf), as in the host build.  key = leaf Morton << 12 | sub-leaf Morton, value = index.
// flags bit 0: outside the root cell, bit 1: non-finite; first_bad: lowest such index.
__global__ __launch_bounds__(256) void k_keys(const double2 *__restrict__ xy, int64_t n, int nside,
                                               uint64_t *__restrict__ key, uint32_t *__restrict__ val,
                                               BuildFacts *__restrict__ facts)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const double x0 = facts->x0, y0 = facts->y0, w = facts->side / (double)nside;
    int *flags = &facts->flags;
    unsigned long long *first_bad = &facts->first_bad;
    const double2 z = xy[i];
    uint32_t c[2] = {0, 0}, f[2] = {0, 0};
    bool bad = false;
    if (!isfinite(z.x) || !isfinite(z.y)) {
        atomicOr(flags, 2);
        bad = true;
    } else {
        for (int d = 0; d < 2; ++d) {
            const double v = ((d ? z.y : z.x) - (d ? y0 : x0)) / w;
            if (!(v >= 0.0) || v > (double)nside) {
                atomicOr(flags, 1);
                bad = true;
                break;
            }
            const int64_t k = (int64_t)floor(v);
            c[d] = (uint32_t)min(k, (int64_t)(nside - 1));
            f[d] = (uint32_t)min((int64_t)floor((v - (double)c[d]) * 64.0), (int64_t)63);
        }
    }
    if (bad) atomicMin(first_bad, (unsigned long long)i);
    key[i] = ((uint64_t)morton_encode(c[0], c[1]) << 12) | morton_encode(f[0], f[1]);
    val[i] = (uint32_t)i;
}

__global__ __launch_bounds__(256) void k_sorted(const uint64_t *__restrict__ key, const uint32_t *__restrict__ val,
                                                 const double2 *__restrict__ xy, int64_t n, int *__restrict__ perm,
                                                 int *__restrict__ leaf_of, double2 *__restrict__ xys)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const uint32_t u = val[i];
    perm[i] = (int)u;
    leaf_of[i] = (int)(key[i] >> 12);
    xys[i] = xy[u];
}

// leaf_start[c] = first sorted slot with leaf >= c, c = 0..nleaf: a binary search per
// leaf (a fill between consecutive occupied leaves would leave one thread to write each
// run of empty leaves, long for clustered particles).
__global__ __launch_bounds__(256) void k_leaf_start(const int *__restrict__ leaf_of, int64_t n, int64_t nleaf,
                                                     int *__restrict__ ls)
{
    const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (c > nleaf) return;
    int64_t lo = 0, hi = n;
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if (leaf_of[mid] < c) lo = mid + 1;
        else hi = mid;
    }
    ls[c] = (int)lo;
}

// Occupancy of every cell of every level (global cell index (4^l - 1)/3 + Morton).
__global__ __launch_bounds__(256) void k_counts(const int *__restrict__ ls, int L, int64_t ncells,
                                                 int *__restrict__ counts)
{
    const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= ncells) return;
    int l = 0;
    while (level_base(l + 1) <= g) ++l;
    const int64_t c = g - level_base(l);
    const int sh = 2 * (L - l);
    counts[g] = ls[(c + 1) << sh] - ls[c << sh];
}

__global__ __launch_bounds__(256) void k_leaf_tiles(const int *__restrict__ ls, int64_t nleaf,
                                                     uint32_t *__restrict__ ntile)
{
    const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (c > nleaf) return;
    ntile[c] = c == nleaf ? 0u : (uint32_t)((ls[c + 1] - ls[c] + 63) / 64);
}

__global__ __launch_bounds__(256) void k_tile_leaf(const uint32_t *__restrict__ tile_start, int64_t nleaf,
                                                    int *__restrict__ tile_leaf)
{
    const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= nleaf) return;
    for (uint32_t t = tile_start[c]; t < tile_start[c + 1]; ++t) tile_leaf[t] = (int)c;
}

// Bounding box of each 64-particle tile in leaf units about the leaf centre, rounded
// outwards to FP32 (as the host build); 16 lanes per tile.
__global__ __launch_bounds__(256) void k_tile_box(const int *__restrict__ tile_leaf,
                                                   const uint32_t *__restrict__ tile_start,
                                                   const int *__restrict__ ls, const double2 *__restrict__ xys,
                                                   int64_t ntiles, double x0, double y0, double w,
                                                   float4 *__restrict__ box)
{
    const int64_t tt = (int64_t)blockIdx.x * 16 + threadIdx.x / 16;
    const int g = threadIdx.x % 16;
    if (tt >= ntiles) return;  // whole groups
    const uint32_t c = (uint32_t)tile_leaf[tt];
    const double cx = x0 + (morton_x(c) + 0.5) * w;
    const double cy = y0 + (morton_y(c) + 0.5) * w;
    const int b = ls[c] + 64 * (int)(tt - tile_start[c]);
    const int e = min(b + 64, ls[c + 1]);
    double xmin = 1e300, ymin = 1e300, xmax = -1e300, ymax = -1e300;
    for (int k = b + g; k < e; k += 16) {
        const double xl = (xys[k].x - cx) / w, yl = (xys[k].y - cy) / w;
        xmin = fmin(xmin, xl);
        xmax = fmax(xmax, xl);
        ymin = fmin(ymin, yl);
        ymax = fmax(ymax, yl);
    }
    for (int o = 8; o >= 1; o >>= 1) {
        xmin = fmin(xmin, __shfl_xor(xmin, o));
        xmax = fmax(xmax, __shfl_xor(xmax, o));
        ymin = fmin(ymin, __shfl_xor(ymin, o));
        ymax = fmax(ymax, __shfl_xor(ymax, o));
    }
    if (g == 0)
        box[tt] = make_float4(nextafterf((float)xmin, -INFINITY), nextafterf((float)ymin, -INFINITY),
                              nextafterf((float)xmax, INFINITY), nextafterf((float)ymax, INFINITY));
}

// Cell lists of levels 2..L grouped by parity class: index k runs over the levels in
// order, inside a level over the classes q = 0..3, inside a class over the cells
// c = 4j + q in increasing order.
__device__ inline void list_cell(int64_t k, int &l, int64_t &c)
{
    l = 2;
    int64_t base = 0;
    while (base + (int64_t(1) << (2 * l)) <= k) {
        base += int64_t(1) << (2 * l);
        ++l;
    }
    const int64_t kk = k - base, quarter = int64_t(1) << (2 * l - 2);
    c = 4 * (kk % quarter) + kk / quarter;
}

__global__ __launch_bounds__(256) void k_list_flags(const int *__restrict__ counts, int64_t nflags,
                                                     uint32_t *__restrict__ flag)
{
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k > nflags) return;
    if (k == nflags) {  // the scan leaves the total there
        flag[k] = 0u;
        return;
    }
    int l;
    int64_t c;
    list_cell(k, l, c);
    flag[k] = counts[level_base(l) + c] > 0 ? 1u : 0u;
}

__global__ __launch_bounds__(256) void k_list_scatter(const int *__restrict__ counts, int64_t nflags,
                                                       const uint32_t *__restrict__ pos, int *__restrict__ lists)
{
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= nflags) return;
    int l;
    int64_t c;
    list_cell(k, l, c);
    if (counts[level_base(l) + c] > 0) lists[pos[k]] = (int)c;
}

// The sizes the host allocates by, from the scanned counts: tiles, cells in the lists (and
// where each class of each level begins), near-field work entries.
__global__ void k_sizes(const uint32_t *__restrict__ tile_start, const uint32_t *__restrict__ pos,
                        const uint32_t *__restrict__ nent, int64_t nleaf, int L, BuildFacts *__restrict__ f)
{
    const int k = threadIdx.x;
    if (k == 0) {
        f->ntiles = tile_start[nleaf];
        f->nlist = L >= 2 ? pos[level_base(L + 1) - level_base(2)] : 0u;
        f->nwork = nent ? nent[nleaf] : 0u;
    }
    if (k >= 8 && k < 4 * (L + 1)) {
        const int l = k / 4, q = k % 4;
        const int64_t quarter = int64_t(1) << (2 * l - 2);
        f->class_off[k] = pos[level_base(l) - level_base(2) + q * quarter];
    }
}

__device__ inline int leaf_count(const int *__restrict__ ls, int nside, int x, int y)
{
    if (x < 0 || y < 0 || x >= nside || y >= nside) return 0;
    const uint32_t c = morton_encode((uint32_t)x, (uint32_t)y);
    return ls[c + 1] - ls[c];
}

// Per leaf: near-field pair sum, occupancy statistics, and the target-centric work
// units (one per 64-particle tile, cost = source steps) with their sort keys.
__global__ __launch_bounds__(256) void k_leaf_stats(const int *__restrict__ ls, int L,
                                                     const uint32_t *__restrict__ tile_start,
                                                     unsigned long long *__restrict__ stats, int4 *__restrict__ units,
                                                     uint64_t *__restrict__ ukey, uint32_t *__restrict__ uval)
{
    const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int nside = 1 << L;
    const int nt = c < (int64_t(1) << (2 * L)) ? ls[c + 1] - ls[c] : 0;
    int64_t nsrc = 0;
    if (nt > 0) {
        const int x = (int)morton_x((uint32_t)c), y = (int)morton_y((uint32_t)c);
        for (int dy = -1; dy <= 1; ++dy)
            for (int dx = -1; dx <= 1; ++dx) nsrc += leaf_count(ls, nside, x + dx, y + dy);
    }
    __shared__ int top[4];
    int most = nt;
    for (int o = 32; o >= 1; o >>= 1) most = max(most, __shfl_xor(most, o));
    if ((threadIdx.x & 63) == 0) top[threadIdx.x >> 6] = most;
    block_add<2>(stats, {(unsigned long long)((int64_t)nt * nsrc), nt > 0 ? 1ull : 0ull});  // (a barrier inside)
    if (threadIdx.x == 0) {
        most = max(max(top[0], top[1]), max(top[2], top[3]));
        if (most > 0) atomicMax(&stats[2], (unsigned long long)most);
    }
    if (nt == 0) return;
    uint32_t tt = tile_start[c];
    for (int c0 = 0; c0 < nt; c0 += 64, ++tt) {
        const int cnt = min(64, nt - c0);
        int logtp = 0;
        while ((1 << logtp) < cnt) ++logtp;
        const int kstride = 64 >> logtp;
        units[tt] = make_int4((int)c, ls[c] + c0, cnt, logtp);
        ukey[tt] = cost_order((uint64_t)((nsrc + kstride - 1) / kstride));  // heaviest first
        uval[tt] = tt;
    }
}

// Non-empty (target, source) cell pairs of the interaction lists, all levels: a thread per
// list entry.
__global__ __launch_bounds__(256) void k_m2l_count(const int *__restrict__ lists, int64_t nlist, int L,
                                                    const BuildFacts *__restrict__ facts,
                                                    const int *__restrict__ counts,
                                                    unsigned long long *__restrict__ stats)
{
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    unsigned long long m = 0;
    if (k < nlist) {
        int l = 2;
        while (l < L && k >= (int64_t)facts->class_off[4 * (l + 1)]) ++l;
        const int n1 = 1 << l;
        const int tx = (int)morton_x((uint32_t)lists[k]), ty = (int)morton_y((uint32_t)lists[k]);
        const int qx = tx & 1, qy = ty & 1;
        for (int dy = -2 - qy; dy <= 3 - qy; ++dy)
            for (int dx = -2 - qx; dx <= 3 - qx; ++dx) {
                if (abs(dx) <= 1 && abs(dy) <= 1) continue;
                const int sx = tx + dx, sy = ty + dy;
                if (sx < 0 || sy < 0 || sx >= n1 || sy >= n1) continue;
                if (counts[level_base(l) + morton_encode((uint32_t)sx, (uint32_t)sy)] > 0) ++m;
            }
    }
    block_add<1>(&stats[3], {m});
}

template <typename T>
__global__ __launch_bounds__(256) void k_gather(const T *__restrict__ src, const uint32_t *__restrict__ idx, int64_t m,
                                                 T *__restrict__ dst)
{
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k < m) dst[k] = src[idx[k]];
}

// Staging slots of the two-pass permutation of the circulations (see pack_kernel):
// sort key of user index u = bucket of its sorted slot.
__global__ __launch_bounds__(256) void k_stage_keys(const int *__restrict__ perm, int64_t n, int shift,
                                                     uint64_t *__restrict__ key, uint32_t *__restrict__ val)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    key[perm[i]] = (uint64_t)(i >> shift);  // the sorted slot of user index perm[i] is i
    val[i] = (uint32_t)i;
}

__global__ __launch_bounds__(256) void k_gpos(const uint32_t *__restrict__ sorted_users, int64_t n,
                                               int *__restrict__ gpos1)
{
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= n) return;
    gpos1[sorted_users[k]] = (int)k;
}

__global__ __launch_bounds__(256) void k_gpos2(const int *__restrict__ gpos1, const int *__restrict__ perm, int64_t n,
                                                int *__restrict__ gpos2)
{
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k < n) gpos2[k] = gpos1[perm[k]];
}

// ---------------------------------------------------------------------------------
// Near-field plan (the mutual form; see build_near_plan_device for its meaning).
// Per leaf: its entries (target-centric units, then the self item, then the items of
// its dense upper neighbours), their costs, the slot mask; then a stable sort by cost.
// ---------------------------------------------------------------------------------
__device__ inline int64_t nch16(int len) { return (len + 15) >> 4; }

__device__ inline int64_t block_steps(int cs, int cr)
{
    const int64_t fs = cs / 64, fr = cr / 64;
    const int rs = cs % 64, rr = cr % 64;
    return 16 * (fs * fr * 4 + fs * nch16(rr) + fr * nch16(rs) + min(nch16(rs), nch16(rr)));
}

// Estimated costs of the entries (a multiple of the steps of 64 pairs that they take).
__device__ inline int log2_lanes(int cnt)
{
    int logtp = 0;
    while ((1 << logtp) < cnt) ++logtp;
    return logtp;
}
__device__ inline int64_t unit_cost(int64_t nsrc, int cnt)
{
    const int kstride = 64 >> log2_lanes(cnt);
    return 2 * ((nsrc + kstride - 1) / kstride);
}
__device__ inline int64_t self_cost(int nt)
{
    const int64_t f = nt / 64;
    const int r = nt % 64;
    return 3 * 16 * (f * (f - 1) / 2 * 4 + f * nch16(r)) + 2 * 16 * (f * 4 + nch16(r));
}

__constant__ int kUp[4][2] = {{1, 0}, {-1, 1}, {0, 1}, {1, 1}};

// A dense leaf's mutual items: item(R, count of R, direction, cost) for itself and for its dense
// upper neighbours.
template <typename Item>
__device__ __forceinline__ void leaf_items(const int *__restrict__ ls, int nside, int64_t c, int nt, int D, Item item)
{
    const int x = (int)morton_x((uint32_t)c), y = (int)morton_y((uint32_t)c);
    item((int)c, nt, 4, self_cost(nt));
    for (int k = 0; k < 4; ++k) {
        const int nr = leaf_count(ls, nside, x + kUp[k][0], y + kUp[k][1]);
        if (nr >= D)
            item((int)morton_encode((uint32_t)(x + kUp[k][0]), (uint32_t)(y + kUp[k][1])), nr,
                 3 * (kUp[k][1] + 1) + (kUp[k][0] + 1), 3 * block_steps(nt, nr));
    }
}

// How an item of this cost between leaves of ns and nr particles is cut (kSplitShare): the tiles
// of the larger leaf in `parts` <= most ranges of `tiles`; one part: not at all.
struct Split {
    int parts, tiles;
};
__device__ inline Split split_of(int64_t cost, int ns, int nr, unsigned long long total, int most)
{
    const int64_t target = max(kSplitLeast, (int64_t)(total / ((unsigned long long)kSplitSimds * kSplitShare)));
    const int na = (max(ns, nr) + 63) / 64;
    if (cost <= 2 * target || na < 2 || most < 2) return Split{1, na};
    const int tiles = (int)max(target * na / cost, (int64_t)max(1, (na + most - 1) / most));
    return Split{(na + tiles - 1) / tiles, tiles};
}

// Sources that the target-centric units of a leaf of nt take, and (mask) the slots its mutual
// items write.
__device__ __forceinline__ int64_t unit_sources(const int *__restrict__ ls, int nside, int64_t c, int nt, int D,
                                                uint32_t &mask)
{
    const int x = (int)morton_x((uint32_t)c), y = (int)morton_y((uint32_t)c);
    int64_t nsrc = 0;
    for (int dy = -1; dy <= 1; ++dy)
        for (int dx = -1; dx <= 1; ++dx) {
            const int ns = leaf_count(ls, nside, x + dx, y + dy);
            if (ns == 0) continue;
            if (nt >= D && ns >= D) mask |= 1u << (3 * (dy + 1) + (dx + 1));
            else nsrc += ns;
        }
    return nsrc;
}

// Per leaf: its mask and units, and the estimated cost of the whole near field.
__global__ __launch_bounds__(256) void k_plan_cost(const int *__restrict__ ls, int L, int D, uint16_t *__restrict__ mask,
                                                   unsigned long long *__restrict__ stats)
{
    const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t nleaf = int64_t(1) << (2 * L);
    const int nside = 1 << L;
    const int nt = c < nleaf ? ls[c + 1] - ls[c] : 0;
    uint32_t m = 0;
    int64_t units = 0, items = 0, pairs = 0, cost = 0;
    if (nt > 0) {
        const int64_t nsrc = unit_sources(ls, nside, c, nt, D, m);
        if (nsrc > 0) {
            m |= 1u << 9;
            units = (nt + 63) / 64;
            cost = (nt / 64) * unit_cost(nsrc, 64) + (nt % 64 ? unit_cost(nsrc, nt % 64) : 0);
        }
        if (nt >= D)
            leaf_items(ls, nside, c, nt, D, [&](int R, int nr, int, int64_t cst) {
                ++items;
                pairs += R == (int)c ? (int64_t)nt * (nt - 1) : 2 * (int64_t)nt * nr;
                cost += cst;
            });
    }
    static_assert(kPlanUnits == 0 && kPlanItems == 1 && kPlanPairs == 2 && kPlanCost == 3, "added together");
    block_add<4>(stats, {(unsigned long long)units, (unsigned long long)items, (unsigned long long)pairs,
                         (unsigned long long)cost});
    if (c < nleaf) mask[c] = (uint16_t)m;
}

// Per leaf: how many entries (nleaf + 1 counts, the last 0); split items, parts and places in the
// parts' sums in all.
__global__ __launch_bounds__(256) void k_plan_count(const int *__restrict__ ls, int L, int D,
                                                     const uint16_t *__restrict__ mask, int most,
                                                     unsigned long long *__restrict__ stats,
                                                     uint32_t *__restrict__ nentries)
{
    const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t nleaf = int64_t(1) << (2 * L);
    const int nt = c < nleaf ? ls[c + 1] - ls[c] : 0;
    const unsigned long long total = stats[kPlanCost];
    uint32_t entries = 0;
    unsigned long long split = 0, parts = 0, sums = 0;
    if (nt > 0) {
        if (mask[c] >> 9) entries = (uint32_t)((nt + 63) / 64);
        if (nt >= D)
            leaf_items(ls, 1 << L, c, nt, D, [&](int, int nr, int, int64_t cost) {
                const Split sp = split_of(cost, nt, nr, total, most);
                entries += sp.parts;
                if (sp.parts == 1) return;
                ++split;
                parts += sp.parts;
                sums += (unsigned long long)sp.parts * min(nt, nr);
            });
    }
    static_assert(kPlanParts == kPlanSplit + 1 && kPlanSums == kPlanSplit + 2, "added together");
    block_add<3>(stats + kPlanSplit, {split, parts, sums});
    if (c <= nleaf) nentries[c] = entries;
}

struct PlanOut {
    int4 *work;
    uint64_t *key;
    uint32_t *val;
    int4 *split, *parts;
};

__global__ __launch_bounds__(256) void k_plan_fill(const int *__restrict__ ls, int L, int D,
                                                    int most, unsigned long long *__restrict__ stats,
                                                    const uint32_t *__restrict__ off, const PlanOut out)
{
    const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= (int64_t(1) << (2 * L))) return;
    const int nside = 1 << L;
    const int nt = ls[c + 1] - ls[c];
    if (nt == 0) return;
    uint32_t m = 0;
    const int64_t nsrc = unit_sources(ls, nside, c, nt, D, m);
    uint32_t o = off[c];
    auto put = [&](int4 e, int64_t cost) {
        out.work[o] = e;
        out.key[o] = cost_order((uint64_t)cost);  // heaviest first
        out.val[o] = o;
        ++o;
    };
    if (nsrc > 0)
        for (int c0 = 0; c0 < nt; c0 += 64) {
            const int cnt = min(64, nt - c0);
            put(make_int4((int)c, ls[c] + c0, cnt, log2_lanes(cnt) | (nt >= D ? 16 : 0)), unit_cost(nsrc, cnt));
        }
    if (nt < D) return;
    const unsigned long long total = stats[kPlanCost];
    leaf_items(ls, nside, c, nt, D, [&](int R, int nr, int ds, int64_t cost) {
        const Split sp = split_of(cost, nt, nr, total, most);
        if (sp.parts == 1) {
            put(make_int4((int)c, R, ds | ((8 - ds) << 4), kMutualItem), cost);
            return;
        }
        // the larger leaf is the one cut
        const bool self = R == (int)c, turn = nt > nr;
        const int S = turn ? R : (int)c, A = turn ? (int)c : R, d = turn ? 8 - ds : ds;
        const int a0 = ls[A], a1 = ls[A + 1], ns = min(nt, nr);
        // (the places are given out in any order: they are addresses, not an order of sums)
        uint32_t at_part = (uint32_t)atomicAdd(&stats[kPlanNext + 1], (unsigned long long)sp.parts);
        uint32_t at_sum = (uint32_t)atomicAdd(&stats[kPlanNext + 2], (unsigned long long)sp.parts * ns);
        out.split[atomicAdd(&stats[kPlanNext], 1ull)] = make_int4(S, d, (int)at_part, sp.parts);
        for (int p = 0; p < sp.parts; ++p) {
            const int first = a0 + 64 * sp.tiles * p, end = min(a1, first + 64 * sp.tiles);
            out.parts[at_part] = make_int4(first, end, (int)at_sum, 0);
            ++at_part;
            at_sum += (uint32_t)ns;
            // (of a leaf with itself a part meets the tiles up to its own)
            const int64_t part_cost = self ? 3 * block_steps(end - a0, end - first) : 3 * block_steps(ns, end - first);
            put(make_int4(S, A, d | ((8 - d) << 4), kMutualItem | ((int)at_part << 9)), part_cost);
        }
    });
}

}  // namespace

namespace {

// A tree array of at least `count` elements from the stream-ordered pool: the one it has
// (taken over from the tree being rebuilt) when that is large enough, else a new one with
// an eighth to spare for the next positions.
template <typename T> hipError_t pool_array(T *&p, int64_t &cap, int64_t count, hipStream_t s)
{
    if (p && cap >= count) return hipSuccess;
    if (p) (void)hipFreeAsync((void *)p, s);
    p = nullptr;
    cap = std::max<int64_t>(count + count / 8, 64);
    const hipError_t e = pool_malloc((void **)&p, (size_t)cap * sizeof(T), s);
    if (e != hipSuccess) cap = 0;
    return e;
}

// The arrays whose sizes n and the depth fix, in one block of the pool (kept from the tree
// being rebuilt, whose n and depth are the same).
hipError_t alloc_slab(fmm_tree *t, hipStream_t s)
{
    if (t->slab) return hipSuccess;
    const size_t n = (size_t)t->n, nleaf = size_t(1) << (2 * t->depth);
    size_t off = 0;
    auto take = [&](size_t bytes) {
        const size_t at = off;
        off += (bytes + 255) / 256 * 256;
        return at;
    };
    const size_t xy = take(n * sizeof(double2)), st1 = take(n * sizeof(double)), perm = take(n * sizeof(int)),
                 g1 = take(n * sizeof(int)), g2 = take(n * sizeof(int)), lo = take(n * sizeof(int)),
                 ls = take((nleaf + 1) * sizeof(int)), ts = take((nleaf + 1) * sizeof(int)),
                 co = take((size_t)level_base(t->depth + 1) * sizeof(int)), ma = take(nleaf * sizeof(uint16_t));
    const hipError_t e = pool_malloc((void **)&t->slab, off, s);
    if (e != hipSuccess) return e;
    char *b = t->slab;
    t->d_xy = (double2 *)(b + xy);
    t->d_st1 = (double *)(b + st1);
    t->d_perm = (int *)(b + perm);
    t->d_gpos1 = (int *)(b + g1);
    t->d_gpos2 = (int *)(b + g2);
    t->d_leaf_of = (int *)(b + lo);
    t->d_leaf_start = (int *)(b + ls);
    t->d_tile_start = (int *)(b + ts);
    t->d_counts = (int *)(b + co);
    t->d_leaf_mask = (uint16_t *)(b + ma);
    return hipSuccess;
}

// Exclusive scan on stream s; *total (device, may be null) receives the sum.
bool scan_on(const uint32_t *in, uint32_t *out, int64_t n, uint32_t *total, hipStream_t s, Status &st)
{
    const int64_t nb = std::max<int64_t>(1, (n + kScanTile - 1) / kScanTile);
    if (nb <= 8) {
        scan_short<<<1, 256, 0, s>>>(in, out, n, total);
        return st.check(hipGetLastError(), "scan launch");
    }
    Buf<uint32_t> sums;
    if (!st.check(sums.alloc(nb, s), "scan workspace")) return false;
    scan_tile_sums<<<(unsigned)nb, 256, 0, s>>>(in, n, sums.p);
    if (nb > kScanSelf) {  // the sums' own scan first; every tile then reads only its own
        if (!scan_on(sums.p, sums.p, nb, nullptr, s, st)) return false;
        scan_add<<<(unsigned)nb, 256, 0, s>>>(in, out, n, sums.p, total);
    } else {
        scan_tiles<<<(unsigned)nb, 256, 0, s>>>(in, out, n, sums.p, total);
    }
    return st.check(hipGetLastError(), "scan launch");
}

}  // namespace

// Exclusive scan of n uint32 (in place allowed); *total_host receives the sum if non-null.
bool scan_exclusive(const uint32_t *in, uint32_t *out, int64_t n, uint32_t *total_host, hipStream_t s, Status &st)
{
    Buf<uint32_t> total;
    if (total_host && !st.check(total.alloc(1, s), "scan workspace")) return false;
    if (!scan_on(in, out, n, total.p, s, st)) return false;
    if (total_host) {
        if (!st.check(hipMemcpyAsync(total_host, total.p, sizeof(uint32_t), hipMemcpyDeviceToHost, s), "scan total") ||
            !st.check(hipStreamSynchronize(s), "scan total"))
            return false;
    }
    return true;
}

// Stable sort of (keys, vals) by the low `bits` bits of the keys.
namespace {

template <int R>
bool radix_passes(Buf<uint64_t> &keys, Buf<uint32_t> &vals, int64_t n, int bits, hipStream_t s, Status &st)
{
    const int nb = (int)((n + 256 * R - 1) / (256 * R));
    Buf<uint64_t> k2;
    Buf<uint32_t> v2, counts;
    if (!st.check(k2.alloc(n, s, keys.kept), "sort workspace") || !st.check(v2.alloc(n, s, vals.kept), "sort workspace") ||
        !st.check(counts.alloc((int64_t)256 * nb + 256, s), "sort workspace"))
        return false;
    uint32_t *totals = counts.p + (int64_t)256 * nb;
    for (int shift = 0; shift < bits; shift += 8) {
        rs_hist<R><<<nb, 256, 0, s>>>(keys.p, n, shift, counts.p, nb);
        rs_scan<<<256, 256, 0, s>>>(counts.p, nb, totals);
        rs_scatter<R><<<nb, 256, 0, s>>>(keys.p, vals.p, k2.p, v2.p, n, shift, counts.p, nb, totals);
        if (!st.check(hipGetLastError(), "sort launch")) return false;
        keys.swap(k2);
        vals.swap(v2);
    }
    return true;
}

}  // namespace

namespace {

bool radix_one(Buf<uint64_t> &keys, Buf<uint32_t> &vals, int64_t n, int bits, hipStream_t s, Status &st)
{
    Buf<uint64_t> k2;
    Buf<uint32_t> v2;
    if (!st.check(k2.alloc(n, s, keys.kept), "sort workspace") || !st.check(v2.alloc(n, s, vals.kept), "sort workspace"))
        return false;
    auto k = n <= 4096 ? rs_one<4> : rs_one<8>;
    k<<<1, 1024, 0, s>>>(keys.p, vals.p, k2.p, v2.p, (int)n, bits);
    if (!st.check(hipGetLastError(), "sort launch")) return false;
    if ((bits + 7) / 8 % 2 == 1) {
        keys.swap(k2);
        vals.swap(v2);
    }
    return true;
}

}  // namespace

bool radix_sort(Buf<uint64_t> &keys, Buf<uint32_t> &vals, int64_t n, int bits, hipStream_t s, Status &st)
{
    if (n <= 1 || bits <= 0) return true;
    if (n <= kOneSort) return radix_one(keys, vals, n, bits, s, st);
    return n <= kSmallSort ? radix_passes<2>(keys, vals, n, bits, s, st) : radix_passes<8>(keys, vals, n, bits, s, st);
}

bool bounding_square(const double2 *xy, int64_t n, hipStream_t s, Status &st, double box[3], bool &nonfinite)
{
    const int nb = (int)std::min<int64_t>(1024, (n + 255) / 256);
    Buf<double4> part;
    Buf<int> flags;
    std::vector<double4> h(nb);
    int hf = 0;
    if (!st.check(part.alloc(nb, s), "bounding square") || !st.check(flags.alloc(1, s), "bounding square") ||
        !st.check(hipMemsetAsync(flags.p, 0, sizeof(int), s), "bounding square"))
        return false;
    k_minmax<<<nb, 256, 0, s>>>(xy, n, part.p, flags.p, 2);
    if (!st.check(hipMemcpyAsync(h.data(), part.p, nb * sizeof(double4), hipMemcpyDeviceToHost, s), "bounding square") ||
        !st.check(hipMemcpyAsync(&hf, flags.p, sizeof(int), hipMemcpyDeviceToHost, s), "bounding square") ||
        !st.check(hipStreamSynchronize(s), "bounding square"))
        return false;
    nonfinite = (hf & 2) != 0;
    double xmin = h[0].x, xmax = h[0].y, ymin = h[0].z, ymax = h[0].w;
    for (int b = 1; b < nb; ++b) {
        xmin = std::min(xmin, h[b].x);
        xmax = std::max(xmax, h[b].y);
        ymin = std::min(ymin, h[b].z);
        ymax = std::max(ymax, h[b].w);
    }
    double side = std::max(xmax - xmin, ymax - ymin);
    if (side <= 0.0) side = 1.0;
    box[0] = xmin;
    box[1] = ymin;
    box[2] = side * (1.0 + 1.0 / 1048576.0);
    return true;
}


// ---------------------------------------------------------------------------------
// Near-field plan of the mutual form (stage 9), from the device leaf offsets (both
// builds use it).  A leaf is dense when it holds at least dense_leaf particles.  Every
// unordered pair of neighbouring dense leaves, and every dense leaf with itself, is one
// mutual item; every other ordered (target leaf, source leaf) pair is evaluated by the
// target-centric units, whose flag makes dense target leaves skip their dense
// neighbours.  leaf_mask[leaf]: bit d (direction d = 3(dy+1) + (dx+1) of a neighbour)
// when the particles' slot d is written, bit 9 when a target-centric unit writes their
// near-field sum.  With the mutual form off the plan is empty and the target-centric
// units cover every pair.
// ---------------------------------------------------------------------------------
namespace {

// Most parts of a split item: 32, but few enough that their sums (which at worst every leaf has
// with five neighbours) stay below some GB.
int most_parts(int64_t n)
{
    if (n > int64_t(1) << 26) return 1;
    return (int)std::min<int64_t>(32, std::max<int64_t>(4, (int64_t(1) << 25) / n));
}

// The plan's counts: entries per leaf (scanned into offsets, nleaf + 1), the leaf masks, and the
// first of plan[] (device, zeroed), see PlanFact.  most: parts of an item.
bool plan_count(fmm_tree *t, Buf<uint32_t> &nent, int most, unsigned long long *plan, hipStream_t s, Status &st)
{
    const int64_t nleaf = int64_t(1) << (2 * t->depth);
    if (!nent.p && !st.check(nent.alloc(nleaf + 1, s), "near-field plan")) return false;
    k_plan_cost<<<grid_for(nleaf, 256), 256, 0, s>>>(t->d_leaf_start, t->depth, t->dense_leaf, t->d_leaf_mask, plan);
    k_plan_count<<<grid_for(nleaf + 1, 256), 256, 0, s>>>(t->d_leaf_start, t->depth, t->dense_leaf, t->d_leaf_mask,
                                                           most, plan, nent.p);
    return scan_on(nent.p, nent.p, nleaf + 1, nullptr, s, st);
}

// The arrays of the split items; none of them if memory does not hold them.
bool part_arrays(fmm_tree *t, const unsigned long long *h, hipStream_t s)
{
    if (pool_array(t->d_split, t->cap_split, (int64_t)h[kPlanSplit], s) == hipSuccess &&
        pool_array(t->d_parts, t->cap_parts, (int64_t)h[kPlanParts], s) == hipSuccess &&
        pool_array(t->d_part_sums, t->cap_part_sums, 3 * (int64_t)h[kPlanSums], s) == hipSuccess)
        return true;
    auto drop = [s](auto *&p, int64_t &cap) {
        if (p) (void)hipFreeAsync((void *)p, s);
        p = nullptr;
        cap = 0;
    };
    drop(t->d_split, t->cap_split);
    drop(t->d_parts, t->cap_parts);
    drop(t->d_part_sums, t->cap_part_sums);
    return false;
}

// The work list of `total` entries, heaviest first, and the parts of the split items; plan as the
// host read it and on the device.  Where the parts' arrays do not fit, the items stay whole.
bool plan_fill(fmm_tree *t, Buf<uint32_t> &nent, uint32_t total, const unsigned long long *h,
               unsigned long long *plan, hipStream_t s, Status &st)
{
    const int64_t nleaf = int64_t(1) << (2 * t->depth);
    int most = most_parts(t->n);
    if (h[kPlanSplit] > 0 && !part_arrays(t, h, s)) {
        most = 1;
        if (!st.check(hipMemsetAsync(plan, 0, kPlanFacts * sizeof(unsigned long long), s), "near-field plan") ||
            !plan_count(t, nent, most, plan, s, st) ||
            !st.check(hipMemcpyAsync(&total, nent.p + nleaf, sizeof total, hipMemcpyDeviceToHost, s), "near-field plan") ||
            !st.check(hipStreamSynchronize(s), "near-field plan"))
            return false;
    }
    Buf<int4> work;
    Buf<uint64_t> key;
    Buf<uint32_t> val;
    if (!st.check(pool_array(t->d_near_work, t->cap_near_work, total, s), "near-field plan") ||
        !st.check(work.alloc(total, s), "near-field plan") || !st.check(key.alloc(total, s), "near-field plan") ||
        !st.check(val.alloc(total, s), "near-field plan"))
        return false;
    k_plan_fill<<<grid_for(nleaf, 256), 256, 0, s>>>(t->d_leaf_start, t->depth, t->dense_leaf, most, plan, nent.p,
                                                      PlanOut{work.p, key.p, val.p, t->d_split, t->d_parts});
    if (!st.check(hipGetLastError(), "near-field plan") || !radix_sort(key, val, total, 8, s, st)) return false;
    k_gather<int4><<<grid_for(total, 256), 256, 0, s>>>(work.p, val.p, total, t->d_near_work);
    t->nnear_work = total;
    t->nsplit = most > 1 ? (int64_t)h[kPlanSplit] : 0;
    t->npart_sums = most > 1 ? (int64_t)h[kPlanSums] : 0;
    return st.check(hipGetLastError(), "near-field plan");
}

void plan_facts(fmm_tree *t, const unsigned long long *plan)
{
    t->nunits_tc = (int64_t)plan[kPlanUnits];
    t->nmut = (int64_t)plan[kPlanItems];
    t->mutual_pairs = (int64_t)plan[kPlanPairs];
}

}  // namespace

int build_near_plan_device(fmm_tree *t, hipStream_t s, std::string &err)
{
    t->nunits_tc = t->nmut = t->nnear_work = t->nsplit = t->npart_sums = t->mutual_pairs = 0;
    if (!t->near_mutual) return FMM_OK;
    Status st;
    auto failed = [&]() {
        err = st.msg;
        return st.code;
    };
    // (an option change: the old plan may be in use)
    if (!st.check(hipDeviceSynchronize(), "near-field plan")) return failed();
    BuildScope scope(s);
    const int64_t nleaf = int64_t(1) << (2 * t->depth);
    Buf<uint32_t> nent;
    Buf<unsigned long long> plan;
    if ((!t->d_leaf_mask &&
         !st.check(pool_malloc((void **)&t->d_leaf_mask, nleaf * sizeof(uint16_t), s), "near-field plan")) ||
        !st.check(plan.alloc(kPlanFacts, s), "near-field plan") ||
        !st.check(hipMemsetAsync(plan.p, 0, kPlanFacts * sizeof(unsigned long long), s), "near-field plan") ||
        !plan_count(t, nent, most_parts(t->n), plan.p, s, st))
        return failed();
    unsigned long long hs[kPlanFacts];
    uint32_t total = 0;
    if (!st.check(hipMemcpyAsync(hs, plan.p, sizeof hs, hipMemcpyDeviceToHost, s), "near-field plan") ||
        !st.check(hipMemcpyAsync(&total, nent.p + nleaf, sizeof total, hipMemcpyDeviceToHost, s), "near-field plan") ||
        !st.check(hipStreamSynchronize(s), "near-field plan"))
        return failed();
    if (!plan_fill(t, nent, total, hs, plan.p, s, st) || !st.check(hipStreamSynchronize(s), "near-field plan")) return failed();
    plan_facts(t, hs);
    return FMM_OK;
}

// ---------------------------------------------------------------------------------
// Stages 1-3 on the device.  xy: device (n, 2) user order.  On success every device
// array of the tree and its host-side counts are set; bad_index receives the first
// offending particle for FMM_EINVAL / FMM_ERANGE.  The host waits three times: for the
// checks, for the sizes of the lists, and at the end.
// ---------------------------------------------------------------------------------
int build_tree_device(fmm_tree *t, const double *xy, const double *root_box, hipStream_t s, std::string &err,
                      int64_t &bad_index, const std::function<void()> &after_checks)
{
    t->pooled = true;
    Status st;
    auto failed = [&]() {
        err = st.msg;
        return st.code;
    };
    const int64_t n = t->n;
    const int L = t->depth;
    const int nside = 1 << L;
    const int64_t nleaf = int64_t(1) << (2 * L);
    const double2 *xy2 = (const double2 *)xy;
    bad_index = -1;
    BuildScope scope(s);
    Buf<BuildFacts> facts;
    BuildFacts h;
    if (!st.check(facts.alloc(1, s), "tree build")) return failed();
    auto read_facts = [&]() {
        return st.check(hipMemcpyAsync(&h, facts.p, sizeof h, hipMemcpyDeviceToHost, s), "tree build") &&
               st.check(hipStreamSynchronize(s), "tree build");
    };
    // Stage 1: root cell (given, or the bounding square).
    constexpr int kBoxNonfinite = 4;
    k_facts<<<1, 1, 0, s>>>(facts.p, root_box ? root_box[0] : 0.0, root_box ? root_box[1] : 0.0,
                            root_box ? root_box[2] : 1.0);
    if (!root_box) {
        const int nb = (int)std::min<int64_t>(1024, (n + 255) / 256);
        Buf<double4> part;
        if (!st.check(part.alloc(nb, s), "bounding square")) return failed();
        k_minmax<<<nb, 256, 0, s>>>(xy2, n, part.p, &facts.p->flags, kBoxNonfinite);
        k_root<<<1, 256, 0, s>>>(part.p, nb, facts.p);
    }
    // Stage 2: keys, then the stable sort by (leaf, sub-leaf key), ties by user index.
    Buf<uint64_t> key;
    Buf<uint32_t> val;
    if (!st.check(key.alloc(n, s), "tree build") || !st.check(val.alloc(n, s), "tree build")) return failed();
    k_keys<<<grid_for(n, 256), 256, 0, s>>>(xy2, n, nside, key.p, val.p, facts.p);
    if (!st.check(hipGetLastError(), "tree build") || !read_facts()) return failed();
    if (h.flags & kBoxNonfinite) {
        err = "non-finite particle position";
        return FMM_EINVAL;
    }
    if (h.flags) {
        bad_index = (int64_t)h.first_bad;
        err = (h.flags & 2) ? "non-finite particle position" : "particle lies outside the root cell";
        return (h.flags & 2) ? FMM_EINVAL : FMM_ERANGE;
    }
    t->x0 = h.x0;
    t->y0 = h.y0;
    t->side = h.side;
    const double w = t->side / (double)nside;
    if (after_checks) after_checks();
    if (!st.check(alloc_slab(t, s), "tree arrays")) return failed();
    if (!radix_sort(key, val, n, 2 * L + 12, s, st)) return failed();
    k_sorted<<<grid_for(n, 256), 256, 0, s>>>(key.p, val.p, xy2, n, t->d_perm, t->d_leaf_of, t->d_xy);
    k_leaf_start<<<grid_for(nleaf + 1, 256), 256, 0, s>>>(t->d_leaf_of, n, nleaf, t->d_leaf_start);
    // Occupancy of all levels; how many tiles, list cells and near-field entries there are.
    const int64_t ncells = level_base(L + 1);
    k_counts<<<grid_for(ncells, 256), 256, 0, s>>>(t->d_leaf_start, L, ncells, t->d_counts);
    uint32_t *tstart = (uint32_t *)t->d_tile_start;
    k_leaf_tiles<<<grid_for(nleaf + 1, 256), 256, 0, s>>>(t->d_leaf_start, nleaf, tstart);
    if (!scan_on(tstart, tstart, nleaf + 1, nullptr, s, st)) return failed();
    const int64_t nflags = L >= 2 ? level_base(L + 1) - level_base(2) : 0;
    Buf<uint32_t> pos, nent;
    if (nflags > 0) {
        if (!st.check(pos.alloc(nflags + 1, s), "cell lists")) return failed();
        k_list_flags<<<grid_for(nflags + 1, 256), 256, 0, s>>>(t->d_counts, nflags, pos.p);
        if (!scan_on(pos.p, pos.p, nflags + 1, nullptr, s, st)) return failed();
    }
    t->nunits_tc = t->nmut = t->nnear_work = t->nsplit = t->npart_sums = t->mutual_pairs = 0;
    if (t->near_mutual && !plan_count(t, nent, most_parts(t->n), facts.p->plan, s, st)) return failed();
    k_sizes<<<1, 64, 0, s>>>(tstart, pos.p, nent.p, nleaf, L, facts.p);
    if (!st.check(hipGetLastError(), "tree build") || !read_facts()) return failed();
    const uint32_t ntiles = h.ntiles;
    t->list_off.assign(L + 1, 0);
    t->list_len.assign(L + 1, 0);
    t->class_off.assign(4 * (L + 1), 0);
    for (int l = 2; l <= L; ++l) {
        const int64_t off = h.class_off[4 * l];
        t->list_off[l] = off;
        for (int q = 0; q < 4; ++q) t->class_off[4 * l + q] = (int64_t)h.class_off[4 * l + q] - off;
        t->list_len[l] = (l < L ? (int64_t)h.class_off[4 * (l + 1)] : (int64_t)h.nlist) - off;
    }
    // Tiles and their boxes, the cell lists, the target-centric units (heaviest first) and
    // the statistics, the near-field plan, the staging slots.
    Buf<int> tile_leaf;
    Buf<int4> units;
    Buf<uint64_t> ukey;
    Buf<uint32_t> uval;
    if (!st.check(pool_array(t->d_tile_box, t->cap_tile_box, ntiles, s), "tile boxes") ||
        !st.check(pool_array(t->d_lists, t->cap_lists, h.nlist, s), "cell lists") ||
        !st.check(pool_array(t->d_units, t->cap_units, ntiles, s), "work units") ||
        !st.check(tile_leaf.alloc(ntiles, s), "tile leaves") || !st.check(units.alloc(ntiles, s), "work units") ||
        !st.check(ukey.alloc(ntiles, s), "work units") || !st.check(uval.alloc(ntiles, s), "work units"))
        return failed();
    k_tile_leaf<<<grid_for(nleaf, 256), 256, 0, s>>>(tstart, nleaf, tile_leaf.p);
    k_tile_box<<<grid_for(ntiles, 16), 256, 0, s>>>(tile_leaf.p, tstart, t->d_leaf_start, t->d_xy, ntiles, t->x0,
                                                     t->y0, w, t->d_tile_box);
    if (nflags > 0)
        k_list_scatter<<<grid_for(nflags, 256), 256, 0, s>>>(t->d_counts, nflags, pos.p, t->d_lists);
    k_leaf_stats<<<grid_for(nleaf, 256), 256, 0, s>>>(t->d_leaf_start, L, tstart, facts.p->stats, units.p, ukey.p,
                                                       uval.p);
    if (h.nlist > 0)
        k_m2l_count<<<grid_for(h.nlist, 256), 256, 0, s>>>(t->d_lists, h.nlist, L, facts.p, t->d_counts,
                                                            facts.p->stats);
    if (!radix_sort(ukey, uval, ntiles, 8, s, st)) return failed();
    k_gather<int4><<<grid_for(ntiles, 256), 256, 0, s>>>(units.p, uval.p, ntiles, t->d_units);
    t->nunits = ntiles;
    if (t->near_mutual && !plan_fill(t, nent, h.nwork, h.plan, facts.p->plan, s, st)) return failed();
    t->stage_shift = stage_shift_of(n);
    if (!build_staging(t->d_perm, n, s, st, t->stage_shift, t->d_gpos1, t->d_gpos2)) return failed();
    if (!st.check(hipGetLastError(), "tree build") || !read_facts()) return failed();
    if (t->near_mutual) plan_facts(t, h.plan);
    t->p2p_pairs = (int64_t)h.stats[0] - n;
    t->nonempty_leaves = (int64_t)h.stats[1];
    t->max_leaf = (int64_t)h.stats[2];
    t->m2l_pairs = (int64_t)h.stats[3];
    return FMM_OK;
}

int stage_shift_of(int64_t n)
{
    int shift = kStageShiftMin;
    while ((((n - 1) >> shift) + 1) > kStageBuckets) ++shift;
    return shift;
}

bool build_staging(const int *perm, int64_t n, hipStream_t s, Status &st, int shift, int *gpos1, int *gpos2)
{
    Buf<uint64_t> key;
    Buf<uint32_t> val;
    if (!st.check(key.alloc(n, s), "staging slots") || !st.check(val.alloc(n, s), "staging slots")) return false;
    k_stage_keys<<<grid_for(n, 256), 256, 0, s>>>(perm, n, shift, key.p, val.p);
    int bits = 0;
    while (((n - 1) >> shift) >> bits) ++bits;  // of the largest bucket number
    if (!radix_sort(key, val, n, bits, s, st)) return false;
    k_gpos<<<grid_for(n, 256), 256, 0, s>>>(val.p, n, gpos1);
    k_gpos2<<<grid_for(n, 256), 256, 0, s>>>(gpos1, perm, n, gpos2);
    return st.check(hipGetLastError(), "staging slots");
}

}  // namespace fmm
