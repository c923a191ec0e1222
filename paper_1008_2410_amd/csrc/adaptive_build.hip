// Stages 1-3 of the adaptive tree on the GPU: keys on the finest grid, the stable sort,
// the cells of all levels at once (a cell splits while it holds more than max_leaf particles
// and lies above max_depth), the same-level neighbours of every cell, the U, V, W and X
// lists, the leaves in sorted order with their 64-particle tiles and tile boxes, and
// the near-field plan.
//
// The arrays equal those of the host build (adaptive.cpp) element for element: cells
// are numbered level by level, in Morton order inside a level; every list is filled by
// the host build's traversal in the host build's order; tile boxes use the same double
// arithmetic (not contracted); and the sorts are stable on the same keys.  So the two
// builds give bit-identical evaluations.
//
// The cells of a level are in Morton order, so the neighbour at (ix + dx, iy + dy) is found by
// a binary search for its Morton code among them.
#include <algorithm>
#include <cmath>
#include <string>
#include <vector>

#include "../../include/fmm2d_adaptive.h"
#include "adaptive_internal.h"
#include "build_prims.h"
#include "fmm_internal.h"

namespace fmm {

namespace {

// Depth of the explicit stack of the U/W walk: it starts with one cell and each step
// that opens a cell replaces it by at most four children, so at most 1 + 3 * 15 entries.
constexpr int kWalkStack = 48;

// Slot of the same-level neighbour at (dx, dy) in {-1, 0, 1}^2 \ {(0, 0)}: the
// directions in the order dy = -1..1, dx = -1..1 with the centre left out (the order in
// which the host build visits neighbours).
__host__ __device__ inline int nb_slot(int dx, int dy)
{
    const int d = 3 * (dy + 1) + (dx + 1);
    return d < 4 ? d : d - 1;
}

__device__ inline int quadrant(const int4 &c, int q) { return q == 0 ? c.x : q == 1 ? c.y : q == 2 ? c.z : c.w; }

// Closed squares of cells a and b ({level, ix, iy, .}) intersect; in units of the
// finest cell.
__device__ inline bool touch(const int4 &a, const int4 &b, int L)
{
    const int64_t sa = int64_t(1) << (L - a.x), sb = int64_t(1) << (L - b.x);
    return a.y * sa <= (b.y + 1) * sb && b.y * sb <= (a.y + 1) * sa && a.z * sa <= (b.z + 1) * sb &&
           b.z * sb <= (a.z + 1) * sa;
}

// Finest-grid cell of every particle (floor binning, clamped at the top edge), as the
// host build: key = its Morton index, value = user index.  flags bit 0: outside the root
// cell, bit 1: non-finite; *first_bad: the lowest such index.
__global__ __launch_bounds__(256) void ak_keys(const double2 *__restrict__ xy, int64_t n, double x0, double y0,
                                                double w, int nside, uint64_t *__restrict__ key,
                                                uint32_t *__restrict__ val, int *__restrict__ flags,
                                                unsigned long long *__restrict__ first_bad)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const double2 z = xy[i];
    uint32_t c[2] = {0, 0};
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
            c[d] = (uint32_t)min((int64_t)floor(v), (int64_t)(nside - 1));
        }
    }
    if (bad) atomicMin(first_bad, (unsigned long long)i);
    key[i] = morton_encode(c[0], c[1]);
    val[i] = (uint32_t)i;
}

__global__ __launch_bounds__(256) void ak_sorted(const uint64_t *__restrict__ key, const uint32_t *__restrict__ val,
                                                  const double2 *__restrict__ xy, int64_t n, int *__restrict__ perm,
                                                  uint32_t *__restrict__ skey, double2 *__restrict__ xs)
{
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= n) return;
    const uint32_t u = val[j];
    perm[j] = (int)u;
    skey[j] = (uint32_t)key[j];
    xs[j] = xy[u];
}

// ---------------------------------------------------------------------------------
// The cells of all levels at once.  In the sorted order a cell is a run of equal key prefixes,
// and it exists when its parent's run is longer than smax; so every particle says by itself
// which cells begin with it, from its key and those smax places away.  (Level by level, each
// level waited for the host to learn how many cells the next one has: 16 levels of 3000001
// clustered particles, 0.9 ms.)
// ---------------------------------------------------------------------------------

// The last level at which two keys lie in one cell.
__device__ inline int common_level(uint32_t a, uint32_t b, int L)
{
    const uint32_t x = a ^ b;
    return x == 0 ? L : L - (33 - __builtin_clz(x)) / 2;
}

// The cells that begin with sorted particle j: levels `first` to `last` (none: last < first),
// those of them below `split` split.
struct CellsAt {
    int first, last, split;
};
__device__ inline CellsAt cells_at(const uint32_t *__restrict__ skey, int64_t n, int64_t j, int smax, int L)
{
    const uint32_t me = skey[j];
    // the run that begins with j is longer than smax down to this level
    const int big = j + smax < n ? common_level(me, skey[j + smax], L) : -1;
    const int split = min(big + 1, L);
    if (j == 0) return CellsAt{0, min(big + 1, L), split};
    const int c = common_level(skey[j - 1], me, L);  // the deepest cell j shares with its predecessor
    if (c == L) return CellsAt{1, 0, 0};
    bool exists = big >= c;  // that cell's run is longer than smax
    if (!exists) {
        if (j >= smax && common_level(skey[j - smax], me, L) >= c) {
            exists = true;
        } else {  // it begins within the smax places before j
            const int shift = 2 * (L - c);
            int64_t lo = j >= smax ? j - smax + 1 : 0, hi = j - 1;
            while (lo < hi) {
                const int64_t mid = (lo + hi) / 2;
                if ((skey[mid] >> shift) == (me >> shift)) hi = mid;
                else lo = mid + 1;
            }
            exists = lo + smax < n && common_level(skey[lo], skey[lo + smax], L) >= c;
        }
    }
    if (!exists) return CellsAt{1, 0, 0};
    return CellsAt{c + 1, max(c + 1, min(big + 1, L)), split};
}

constexpr int kLevels = 32;  // counters per kind: cells, split cells

// How many cells begin with each particle, and the cells and split cells of every level.
__global__ __launch_bounds__(256) void ak_cell_count(const uint32_t *__restrict__ skey, int64_t n, int smax, int L,
                                                     uint32_t *__restrict__ ncells,
                                                     unsigned long long *__restrict__ levels)
{
    __shared__ unsigned int h[2 * kLevels];
    if (threadIdx.x < 2 * kLevels) h[threadIdx.x] = 0;
    __syncthreads();
    for (int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x; j < n; j += (int64_t)gridDim.x * 256) {
        const CellsAt c = cells_at(skey, n, j, smax, L);
        ncells[j] = (uint32_t)(c.last - c.first + 1);
        for (int l = c.first; l <= c.last; ++l) {
            atomicAdd(&h[l], 1u);
            if (l < c.split) atomicAdd(&h[kLevels + l], 1u);
        }
    }
    __syncthreads();
    if (threadIdx.x < 2 * kLevels && h[threadIdx.x]) atomicAdd(&levels[threadIdx.x], (unsigned long long)h[threadIdx.x]);
}

// The cells in the order of their first particles: sort key = level, value = first particle.
__global__ __launch_bounds__(256) void ak_cell_fill(const uint32_t *__restrict__ skey, int64_t n, int smax, int L,
                                                    const uint32_t *__restrict__ off, uint64_t *__restrict__ key,
                                                    uint32_t *__restrict__ val)
{
    const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (j >= n) return;
    const CellsAt c = cells_at(skey, n, j, smax, L);
    uint32_t o = off[j];
    for (int l = c.first; l <= c.last; ++l, ++o) {
        key[o] = (uint64_t)l;
        val[o] = (uint32_t)j;
    }
}

struct LevelOffsets {
    int at[kLevels + 1];
};

// The cells in level order (and Morton order inside a level) from their first particles: square,
// leaf flag, range, parent, the parent's child entry (child filled with -1 before), and code,
// the cell's place in the Morton order of its level.
__global__ __launch_bounds__(256) void ak_cells(const uint32_t *__restrict__ skey, int64_t n, int smax, int L, int K,
                                                const LevelOffsets off, const uint32_t *__restrict__ start,
                                                int4 *__restrict__ cell, int2 *__restrict__ range,
                                                int *__restrict__ parent, int4 *__restrict__ child,
                                                uint32_t *__restrict__ code)
{
    const int k = blockIdx.x * 256 + threadIdx.x;
    if (k >= K) return;
    int l = 0;
    while (k >= off.at[l + 1]) ++l;
    const int64_t j = start[k];
    const int shift = 2 * (L - l);
    const uint32_t me = skey[j], pre = shift < 32 ? me >> shift : 0u;
    const bool split = l < L && j + smax < n && common_level(me, skey[j + smax], L) >= l;
    // one past the run: within smax places of j unless the cell is split or of the last level
    int64_t lo = j + 1, hi = split || l == L ? n : min(n, j + smax);
    while (lo < hi) {
        const int64_t mid = (lo + hi) / 2;
        if ((shift < 32 ? skey[mid] >> shift : 0u) == pre) lo = mid + 1;
        else hi = mid;
    }
    cell[k] = make_int4(l, (int)morton_x(pre), (int)morton_y(pre), split ? 0 : 1);
    range[k] = make_int2((int)j, (int)(lo - j));
    code[k] = pre;
    int P = -1;
    if (l > 0) {  // the last cell of the level above that begins at or before j
        int a = off.at[l - 1], b = off.at[l] - 1;
        while (a < b) {
            const int mid = (a + b + 1) / 2;
            if (start[mid] <= (uint32_t)j) a = mid;
            else b = mid - 1;
        }
        P = a;
        ((int *)(child + P))[pre & 3u] = k;
    }
    parent[k] = P;
}

// Same-level neighbours of every cell (slot order of nb_slot, -1 where there is no cell).
__global__ __launch_bounds__(256) void ak_neighbours(const int4 *__restrict__ cell, const uint32_t *__restrict__ code,
                                                     int K, const LevelOffsets off, int *__restrict__ coll)
{
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t k = t >> 3;
    if (k >= K) return;
    const int slot = (int)(t & 7), d = slot < 4 ? slot : slot + 1;
    const int4 c = cell[k];
    const int nx = c.y + d % 3 - 1, ny = c.z + d / 3 - 1, nside = 1 << c.x;
    int r = -1;
    if (nx >= 0 && ny >= 0 && nx < nside && ny < nside) {
        const uint32_t want = (uint32_t)morton_encode((uint32_t)nx, (uint32_t)ny);
        int a = off.at[c.x], b = off.at[c.x + 1];
        while (a < b) {
            const int mid = (a + b) / 2;
            if (code[mid] < want) a = mid + 1;
            else b = mid;
        }
        if (a < off.at[c.x + 1] && code[a] == want) r = a;
    }
    coll[t] = r;
}

// V list of every cell: children of the parent's neighbours that do not touch it.
// Counting pass (FILL false, K + 1 counts with the last 0) and filling pass.
template <bool FILL>
__global__ __launch_bounds__(256) void ak_vlist(const int4 *__restrict__ cell, const int *__restrict__ parent,
                                                 const int4 *__restrict__ child, const int *__restrict__ coll, int K,
                                                 uint32_t *__restrict__ cnt, const int *__restrict__ off,
                                                 int *__restrict__ idx)
{
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k > K) return;
    if (k == K) {
        if (!FILL) cnt[K] = 0;
        return;
    }
    const int P = parent[k];
    int nv = 0;
    const int o = FILL ? off[k] : 0;
    if (P >= 0) {
        const int4 ck = cell[k];
        for (int j = 0; j < 8; ++j) {
            const int PN = coll[(int64_t)P * 8 + j];
            if (PN < 0) continue;
            const int4 ch = child[PN];
            for (int q = 0; q < 4; ++q) {
                const int d = quadrant(ch, q);
                if (d < 0) continue;
                const int4 cd = cell[d];
                if (abs(cd.y - ck.y) > 1 || abs(cd.z - ck.z) > 1) {
                    if (FILL) idx[o + nv] = d;
                    ++nv;
                }
            }
        }
    }
    if (!FILL) cnt[k] = (uint32_t)nv;
}

// U and W lists of every leaf k: k itself; then, below each same-level neighbour, the
// leaves that touch k (U) and the cells that do not touch k while their parents do (W),
// depth first with quadrants ascending; then the coarser leaves that touch k among the
// neighbours of its ancestors, nearest ancestor first.  W entries carry their owner.
template <bool FILL>
__global__ __launch_bounds__(256) void ak_uwlist(const int4 *__restrict__ cell, const int *__restrict__ parent,
                                                  const int4 *__restrict__ child, const int *__restrict__ coll, int K,
                                                  int L, uint32_t *__restrict__ ucnt, uint32_t *__restrict__ wcnt,
                                                  const int *__restrict__ uoff, const int *__restrict__ woff,
                                                  int *__restrict__ uidx, int *__restrict__ widx,
                                                  uint32_t *__restrict__ wown, int *__restrict__ err)
{
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k > K) return;
    if (k == K) {
        if (!FILL) ucnt[K] = wcnt[K] = 0;
        return;
    }
    const int4 ck = cell[k];
    if (!ck.w) {
        if (!FILL) ucnt[k] = wcnt[k] = 0;
        return;
    }
    int nu = 0, nw = 0;
    const int uo = FILL ? uoff[k] : 0, wo = FILL ? woff[k] : 0;
    if (FILL) uidx[uo] = k;
    ++nu;
    int st[kWalkStack];
    for (int j = 0; j < 8; ++j) {
        const int C = coll[(int64_t)k * 8 + j];
        if (C < 0) continue;
        int sp = 0;
        st[sp++] = C;
        while (sp > 0) {
            const int d = st[--sp];
            const int4 cd = cell[d];
            if (!touch(cd, ck, L)) {
                if (FILL) {
                    widx[wo + nw] = d;
                    wown[wo + nw] = (uint32_t)k;
                }
                ++nw;
                continue;
            }
            if (cd.w) {
                if (FILL) uidx[uo + nu] = d;
                ++nu;
                continue;
            }
            if (sp + 4 > kWalkStack) {  // cannot happen for depth <= 15; reported, never overrun
                atomicOr(err, 1);
                break;
            }
            const int4 ch = child[d];
            if (ch.w >= 0) st[sp++] = ch.w;
            if (ch.z >= 0) st[sp++] = ch.z;
            if (ch.y >= 0) st[sp++] = ch.y;
            if (ch.x >= 0) st[sp++] = ch.x;
        }
    }
    for (int a = parent[k]; a >= 0; a = parent[a])
        for (int j = 0; j < 8; ++j) {
            const int C = coll[(int64_t)a * 8 + j];
            if (C < 0) continue;
            const int4 cc = cell[C];
            if (cc.w && touch(cc, ck, L)) {
                if (FILL) uidx[uo + nu] = C;
                ++nu;
            }
        }
    if (!FILL) {
        ucnt[k] = (uint32_t)nu;
        wcnt[k] = (uint32_t)nw;
    }
}

// X list counts: X(d) holds every a with d in W(a).
__global__ __launch_bounds__(256) void ak_xcount(const int *__restrict__ widx, int64_t nw, uint32_t *__restrict__ xcnt)
{
    const int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (u < nw) atomicAdd(&xcnt[widx[u]], 1u);
}

__global__ __launch_bounds__(256) void ak_xkeys(const int *__restrict__ widx, int64_t nw, uint64_t *__restrict__ key)
{
    const int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (u < nw) key[u] = (uint64_t)widx[u];
}

// First sorted slot of every leaf gets flag 1 (flag zeroed beforehand).
__global__ __launch_bounds__(256) void ak_leaf_marks(const int4 *__restrict__ cell, const int2 *__restrict__ range, int K,
                                                      uint32_t *__restrict__ flag)
{
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k < K && cell[k].w) flag[range[k].x] = 1;
}

// Leaf index (position in sorted order) of every leaf.
__global__ __launch_bounds__(256) void ak_leaf_index(const int4 *__restrict__ cell, const int2 *__restrict__ range,
                                                      int K, const uint32_t *__restrict__ e,
                                                      int *__restrict__ leaf_index, int *__restrict__ leaves,
                                                      int *__restrict__ leaf_start)
{
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= K) return;
    const int4 c = cell[k];
    if (!c.w) {
        leaf_index[k] = -1;
        return;
    }
    const int first = range[k].x;
    const int li = (int)e[first];
    leaf_index[k] = li;
    leaves[li] = k;
    leaf_start[li] = first;
}

// Leaf of every sorted particle: the leaf whose first slot is the last flagged slot <= j.
__global__ __launch_bounds__(256) void ak_leaf_of(const uint32_t *__restrict__ flag, const uint32_t *__restrict__ e,
                                                   const int *__restrict__ leaves, int64_t n, int *__restrict__ leaf_of)
{
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j < n) leaf_of[j] = leaves[e[j] + flag[j] - 1];
}

__global__ void ak_set(int *p, int v) { *p = v; }

// Tiles per leaf (NL + 1 entries, the last 0).
__global__ __launch_bounds__(256) void ak_leaf_ntiles(const int *__restrict__ leaves, const int2 *__restrict__ range,
                                                       int NL, uint32_t *__restrict__ nt)
{
    const int li = blockIdx.x * blockDim.x + threadIdx.x;
    if (li > NL) return;
    nt[li] = li == NL ? 0u : (uint32_t)((range[leaves[li]].y + 63) / 64);
}

// First tile of every leaf cell (tile_start zeroed beforehand) and the leaf of every tile.
__global__ __launch_bounds__(256) void ak_tiles(const int *__restrict__ leaves, const int *__restrict__ leaf_tile, int NL,
                                                 int *__restrict__ tile_start, int *__restrict__ tile_leaf)
{
    const int li = blockIdx.x * blockDim.x + threadIdx.x;
    if (li >= NL) return;
    const int t0 = leaf_tile[li], t1 = leaf_tile[li + 1];
    tile_start[leaves[li]] = t0;
    for (int t = t0; t < t1; ++t) tile_leaf[t] = li;
}

// Box of every tile: {xmin, ymin, xmax, ymax} relative to (x0, y0), and in leaf widths
// about the leaf centre rounded outwards to FP32; the host build's arithmetic, with
// no fused multiply-adds.
__global__ __launch_bounds__(256) void ak_tile_box(const int *__restrict__ tile_leaf, const int *__restrict__ leaves,
                                                    const int *__restrict__ leaf_tile, const int4 *__restrict__ cell,
                                                    const int2 *__restrict__ range, const double2 *__restrict__ xs,
                                                    int64_t ntiles, double x0, double y0, double side,
                                                    double4 *__restrict__ box, float4 *__restrict__ box_leaf)
{
#pragma clang fp contract(off)
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= ntiles) return;
    const int li = tile_leaf[t];
    const int k = leaves[li];
    const int4 c = cell[k];
    const int2 r = range[k];
    const int b = r.x + 64 * (int)(t - leaf_tile[li]);
    const int e = min(b + 64, r.x + r.y);
    const double wl = side / (double)(int64_t(1) << c.x);
    const double cx = x0 + (c.y + 0.5) * wl, cy = y0 + (c.z + 0.5) * wl;
    double4 bx = make_double4(1e300, 1e300, -1e300, -1e300), bl = bx;
    for (int j = b; j < e; ++j) {
        const double2 z = xs[j];
        const double x = z.x - x0, y = z.y - y0;
        bx.x = x < bx.x ? x : bx.x;
        bx.y = y < bx.y ? y : bx.y;
        bx.z = bx.z < x ? x : bx.z;
        bx.w = bx.w < y ? y : bx.w;
        const double xl = (z.x - cx) / wl, yl = (z.y - cy) / wl;
        bl.x = xl < bl.x ? xl : bl.x;
        bl.y = yl < bl.y ? yl : bl.y;
        bl.z = bl.z < xl ? xl : bl.z;
        bl.w = bl.w < yl ? yl : bl.w;
    }
    box[t] = bx;
    box_leaf[t] = make_float4(nextafterf((float)bl.x, -INFINITY), nextafterf((float)bl.y, -INFINITY),
                              nextafterf((float)bl.z, INFINITY), nextafterf((float)bl.w, INFINITY));
}

// Statistics gathered by the plan's counting pass.
enum { kStPairs = 0, kStMutualPairs, kStMutualItems, kStUnits, kStCount };

// Near-field plan, per leaf in sorted order: target-centric units (one per 64-particle
// tile) when some of U is left to them, then for a dense leaf its mutual item with
// itself and with each dense same-level leaf at (1, 0), (-1, 1), (0, 1), (1, 1); the slot
// mask of every leaf.  Counting pass (NL + 1 counts, the last 0; statistics) and
// filling pass (entries, their order keys, and the identity to sort with them).
template <bool FILL>
__global__ __launch_bounds__(256) void ak_plan(const int *__restrict__ leaves, const int *__restrict__ leaf_index, int NL,
                                                const int4 *__restrict__ cell, const int2 *__restrict__ range,
                                                const int *__restrict__ coll, const int *__restrict__ u_off,
                                                const int *__restrict__ u_idx, int D, uint32_t *__restrict__ cnt,
                                                const int *__restrict__ off, int4 *__restrict__ work,
                                                uint64_t *__restrict__ key, uint32_t *__restrict__ order,
                                                uint16_t *__restrict__ mask, unsigned long long *__restrict__ stats)
{
    const int li = blockIdx.x * blockDim.x + threadIdx.x;
    if (FILL && li >= NL) return;
    const bool valid = li < NL;  // the counting pass keeps its wavefronts whole for the sums
    const int k = valid ? leaves[li] : 0;
    const int4 c = cell[k];
    const int2 r = valid ? range[k] : make_int2(0, 0);
    const bool dense = r.y >= D;
    uint32_t m = 0;
    int64_t nsrc = 0, usum = 0;
    for (int u = valid ? u_off[k] : 0, ue = valid ? u_off[k + 1] : 0; u < ue; ++u) {
        const int S = u_idx[u];
        const int4 cs = cell[S];
        const int ns = range[S].y;
        usum += ns;
        if (dense && ns >= D && cs.x == c.x)
            m |= 1u << (3 * (cs.z - c.z + 1) + (cs.y - c.y + 1));
        else
            nsrc += ns;
    }
    int ne = 0;
    const int o = FILL ? off[li] : 0;
    auto put = [&](int4 item, int64_t cst) {
        if (FILL) {
            work[o + ne] = item;
            key[o + ne] = cost_order((uint64_t)cst);  // heaviest first
            order[o + ne] = (uint32_t)(o + ne);
        }
        ++ne;
    };
    int64_t units = 0, items = 0, mp = 0;
    if (nsrc > 0) {
        m |= 1u << 9;
        for (int b = r.x; b < r.x + r.y; b += 64) {
            const int len = min(64, r.x + r.y - b);
            put(make_int4(k, b, len, at_log2_lanes(len) | (dense ? 16 : 0)), at_unit_cost(nsrc, len));
            ++units;
        }
    }
    if (dense) {
        put(make_int4(li, li, 4 | (4 << 4), kMutualItem | (c.x << 9)), at_self_cost(r.y));
        ++items;
        mp += (int64_t)r.y * (r.y - 1);
        const int up[4][2] = {{1, 0}, {-1, 1}, {0, 1}, {1, 1}};
        for (int q = 0; q < 4; ++q) {
            const int R = coll[(int64_t)k * 8 + nb_slot(up[q][0], up[q][1])];
            if (R < 0 || !cell[R].w || range[R].y < D) continue;
            const int ds = 3 * (up[q][1] + 1) + (up[q][0] + 1);
            put(make_int4(li, leaf_index[R], ds | ((8 - ds) << 4), kMutualItem | (c.x << 9)),
                3 * at_pair_steps(r.y, range[R].y));
            ++items;
            mp += 2 * (int64_t)r.y * range[R].y;
        }
    }
    if constexpr (!FILL) {
        if (li <= NL) cnt[li] = (uint32_t)ne;  // 0 at NL
        if (valid) mask[k] = (uint16_t)m;
        unsigned long long v[kStCount];
        v[kStPairs] = (unsigned long long)((int64_t)r.y * usum - r.y);
        v[kStMutualPairs] = (unsigned long long)mp;
        v[kStMutualItems] = (unsigned long long)items;
        v[kStUnits] = (unsigned long long)units;
        block_add<kStCount>(stats, v);
    }
}

__global__ __launch_bounds__(256) void ak_gather_work(const int4 *__restrict__ src, const uint32_t *__restrict__ order,
                                                       int64_t nwork, int4 *__restrict__ dst)
{
    const int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (u < nwork) dst[u] = src[order[u]];
}

// Flags of the leaves of level >= 2 (multipoles from particles) and of the split cells
// of level >= 2 (multipoles from children); K + 1 entries, the last 0.
__global__ __launch_bounds__(256) void ak_cell_flags(const int4 *__restrict__ cell, int K, uint32_t *__restrict__ fleaf,
                                                      uint32_t *__restrict__ finner)
{
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k > K) return;
    if (k == K) {
        fleaf[K] = finner[K] = 0;
        return;
    }
    const int4 c = cell[k];
    fleaf[k] = c.w && c.x >= 2;
    finner[k] = !c.w && c.x >= 2;
}

__global__ __launch_bounds__(256) void ak_compact(const uint32_t *__restrict__ flag, const uint32_t *__restrict__ pos,
                                                   int K, int *__restrict__ out)
{
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k < K && flag[k]) out[pos[k]] = k;
}

// Adjoint near-field units, one per 64-particle tile of every leaf (leaf index li in
// sorted order; tile t = leaf_tile[li] + tile within the leaf): {leaf cell, first, count,
// log2 TP}, cost over all of U(leaf) as for the forward target-centric units.
__global__ __launch_bounds__(256) void ak_adj_units(const int *__restrict__ leaf_start, const int *__restrict__ leaf_of,
                                                     const int *__restrict__ leaf_tile, int NL,
                                                     const int2 *__restrict__ range, const int *__restrict__ u_off,
                                                     const int *__restrict__ u_idx, int4 *__restrict__ units,
                                                     uint64_t *__restrict__ key, uint32_t *__restrict__ order)
{
    const int li = blockIdx.x * blockDim.x + threadIdx.x;
    if (li >= NL) return;
    const int k = leaf_of[leaf_start[li]];
    const int2 r = range[k];
    int64_t usum = 0;
    for (int e = u_off[k]; e < u_off[k + 1]; ++e) usum += range[u_idx[e]].y;
    int t = leaf_tile[li];
    for (int b = r.x; b < r.x + r.y; b += 64, ++t) {
        const int len = min(64, r.x + r.y - b);
        units[t] = make_int4(k, b, len, at_log2_lanes(len));
        key[t] = cost_order((uint64_t)at_unit_cost(usum, len));  // heaviest first
        order[t] = (uint32_t)t;
    }
}

template <typename T>
bool alloc_to(T *&p, int64_t count, hipStream_t s, Status &st, const char *what)
{
    return st.check(build_alloc((void **)&p, (size_t)std::max<int64_t>(count, 1) * sizeof(T), s), what);
}

bool read_back(void *dst, const void *src, size_t bytes, hipStream_t s, Status &st)
{
    return st.check(hipMemcpyAsync(dst, src, bytes, hipMemcpyDeviceToHost, s), "adaptive tree build") &&
           st.check(hipStreamSynchronize(s), "adaptive tree build");
}

int bits_for(uint64_t v)
{
    int b = 0;
    while (b < 64 && (v >> b) != 0) ++b;
    return b;
}

}  // namespace

int build_atree_device(fmm_atree *t, const double *xy, const double *root_box, hipStream_t s, std::string &err,
                       int64_t &bad_index)
{
    t->pooled = true;
    Status st;
    auto failed = [&]() {
        err = st.msg;
        return st.code;
    };
    bad_index = -1;
    const int64_t n = t->n;
    const int L = t->max_depth;
    const int smax = t->max_leaf;
    const double2 *xy2 = (const double2 *)xy;
    AtreeDev &d = t->d;
    BuildScope scope(s);

    // Stage 1: root cell.
    if (root_box) {
        t->x0 = root_box[0];
        t->y0 = root_box[1];
        t->side = root_box[2];
    } else {
        double box[3];
        bool nonfinite = false;
        if (!bounding_square(xy2, n, s, st, box, nonfinite)) return failed();
        if (nonfinite) {
            err = "non-finite particle position";
            return FMM_EINVAL;
        }
        t->x0 = box[0];
        t->y0 = box[1];
        t->side = box[2];
    }
    // Stage 2: keys on the finest grid and the stable sort by key (ties by user index).
    const int nside = 1 << L;
    const double w = t->side / (double)nside;
    Buf<uint64_t> key;
    Buf<uint32_t> val, skey;
    Buf<int> flags;
    Buf<unsigned long long> first_bad;
    if (!st.check(key.alloc(n, s), "adaptive tree build") || !st.check(val.alloc(n, s), "adaptive tree build") ||
        !st.check(skey.alloc(n, s), "adaptive tree build") || !st.check(flags.alloc(1, s), "adaptive tree build") ||
        !st.check(first_bad.alloc(1, s), "adaptive tree build") ||
        !st.check(hipMemsetAsync(flags.p, 0, sizeof(int), s), "adaptive tree build") ||
        !st.check(hipMemsetAsync(first_bad.p, 0xff, sizeof(unsigned long long), s), "adaptive tree build"))
        return failed();
    ak_keys<<<grid_for(n, 256), 256, 0, s>>>(xy2, n, t->x0, t->y0, w, nside, key.p, val.p, flags.p, first_bad.p);
    {
        int hf = 0;
        unsigned long long hb = 0;
        if (!st.check(hipMemcpyAsync(&hf, flags.p, sizeof(int), hipMemcpyDeviceToHost, s), "adaptive tree build") ||
            !read_back(&hb, first_bad.p, sizeof hb, s, st))
            return failed();
        if (hf) {
            bad_index = (int64_t)hb;
            err = (hf & 2) ? "non-finite particle position" : "particle lies outside the root cell";
            return (hf & 2) ? FMM_EINVAL : FMM_ERANGE;
        }
    }
    if (!radix_sort(key, val, n, 2 * L, s, st)) return failed();
    if (!alloc_to(d.perm, n, s, st, "permutation") || !alloc_to(d.xy, n, s, st, "sorted positions") ||
        !alloc_to(d.leaf_of, n, s, st, "leaf of each particle"))
        return failed();
    ak_sorted<<<grid_for(n, 256), 256, 0, s>>>(key.p, val.p, xy2, n, d.perm, skey.p, d.xy);

    // Stage 3a: cells.
    Buf<unsigned long long> levels;
    Buf<uint32_t> cfirst, code;
    Buf<uint64_t> clevel;
    Buf<int> coll;
    if (!st.check(levels.alloc(2 * kLevels, s), "adaptive tree build") ||
        !st.check(hipMemsetAsync(levels.p, 0, 2 * kLevels * sizeof(unsigned long long), s), "adaptive tree build"))
        return failed();
    ak_cell_count<<<std::min<unsigned>(grid_for(n, 256), 1024), 256, 0, s>>>(skey.p, n, smax, L, val.p, levels.p);
    unsigned long long hl[2 * kLevels];
    if (!scan_exclusive(val.p, val.p, n, nullptr, s, st) || !read_back(hl, levels.p, sizeof hl, s, st)) return failed();
    LevelOffsets off{};
    int64_t total = 0, splits = 0;
    int deepest = 0;
    t->inner_off.assign(L + 2, 0);
    t->level_off.assign(L + 2, 0);
    for (int l = 0; l <= L; ++l) {
        total += (int64_t)hl[l];
        splits += (int64_t)hl[kLevels + l];
        if (total >= (int64_t(1) << 31)) {
            err = "adaptive tree: too many cells";
            return FMM_ENOMEM;
        }
        if (hl[l] > 0) deepest = l;
        t->level_off[l + 1] = (int)total;
        t->inner_off[l + 1] = t->inner_off[l] + (l >= 2 ? (int)hl[kLevels + l] : 0);
    }
    for (int l = 0; l <= kLevels; ++l) off.at[l] = l <= L + 1 ? t->level_off[l] : (int)total;
    const int K = (int)total;
    const uint32_t NL = (uint32_t)(total - splits);
    t->ncells = K;
    if (!st.check(cfirst.alloc(K, s), "adaptive tree cells") || !st.check(clevel.alloc(K, s), "adaptive tree cells") ||
        !st.check(code.alloc(K, s), "adaptive tree cells") || !st.check(coll.alloc(8 * (int64_t)K, s), "adaptive tree cells") ||
        !alloc_to(d.cell, K, s, st, "adaptive tree cells") || !alloc_to(d.range, K, s, st, "adaptive tree cells") ||
        !alloc_to(d.parent, K, s, st, "adaptive tree cells") || !alloc_to(d.child, K, s, st, "adaptive tree cells") ||
        !st.check(hipMemsetAsync(d.child, 0xff, (size_t)K * sizeof(int4), s), "adaptive tree cells"))
        return failed();
    ak_cell_fill<<<grid_for(n, 256), 256, 0, s>>>(skey.p, n, smax, L, val.p, clevel.p, cfirst.p);
    if (!radix_sort(clevel, cfirst, K, 8, s, st)) return failed();
    ak_cells<<<grid_for(K, 256), 256, 0, s>>>(skey.p, n, smax, L, K, off, cfirst.p, d.cell, d.range, d.parent, d.child,
                                              code.p);
    ak_neighbours<<<grid_for(8 * (int64_t)K, 256), 256, 0, s>>>(d.cell, code.p, K, off, coll.p);
    if (!st.check(hipGetLastError(), "adaptive tree build")) return failed();

    // Stage 3b: lists.
    Buf<int> werr;
    Buf<uint32_t> ucnt, wcnt, vcnt;
    if (!st.check(werr.alloc(1, s), "adaptive tree build") ||
        !st.check(hipMemsetAsync(werr.p, 0, sizeof(int), s), "adaptive tree build") ||
        !st.check(ucnt.alloc(K + 1, s, true), "adaptive tree lists") || !st.check(wcnt.alloc(K + 1, s, true), "adaptive tree lists") ||
        !st.check(vcnt.alloc(K + 1, s, true), "adaptive tree lists"))
        return failed();
    ak_vlist<false><<<grid_for(K + 1, 256), 256, 0, s>>>(d.cell, d.parent, d.child, coll.p, K, vcnt.p, nullptr,
                                                         nullptr);
    ak_uwlist<false><<<grid_for(K + 1, 256), 256, 0, s>>>(d.cell, d.parent, d.child, coll.p, K, L, ucnt.p, wcnt.p,
                                                          nullptr, nullptr, nullptr, nullptr, nullptr, werr.p);
    uint32_t nv = 0, nu = 0, nw = 0;
    if (!scan_exclusive(vcnt.p, vcnt.p, K + 1, nullptr, s, st) || !scan_exclusive(ucnt.p, ucnt.p, K + 1, nullptr, s, st) ||
        !scan_exclusive(wcnt.p, wcnt.p, K + 1, nullptr, s, st) ||
        !st.check(hipMemcpyAsync(&nv, vcnt.p + K, sizeof nv, hipMemcpyDeviceToHost, s), "adaptive tree lists") ||
        !st.check(hipMemcpyAsync(&nu, ucnt.p + K, sizeof nu, hipMemcpyDeviceToHost, s), "adaptive tree lists") ||
        !read_back(&nw, wcnt.p + K, sizeof nw, s, st))
        return failed();
    // the scanned counts are the CSR offsets (totals below 2^31)
    d.v_off = (int *)vcnt.release();
    d.u_off = (int *)ucnt.release();
    d.w_off = (int *)wcnt.release();
    Buf<uint32_t> wown;
    if (!alloc_to(d.v_idx, nv, s, st, "V list") || !alloc_to(d.u_idx, nu, s, st, "U list") ||
        !alloc_to(d.w_idx, nw, s, st, "W list") || !st.check(wown.alloc(nw, s, true), "W list"))
        return failed();
    ak_vlist<true><<<grid_for(K + 1, 256), 256, 0, s>>>(d.cell, d.parent, d.child, coll.p, K, nullptr, d.v_off,
                                                        d.v_idx);
    ak_uwlist<true><<<grid_for(K + 1, 256), 256, 0, s>>>(d.cell, d.parent, d.child, coll.p, K, L, nullptr, nullptr,
                                                         d.u_off, d.w_off, d.u_idx, d.w_idx, wown.p, werr.p);
    // X: the W entries (in owner order) stably sorted by the cell they name.
    {
        Buf<uint32_t> xcnt;
        Buf<uint64_t> xkey;
        if (!st.check(xcnt.alloc(K + 1, s, true), "X list") ||
            !st.check(hipMemsetAsync(xcnt.p, 0, (K + 1) * sizeof(uint32_t), s), "X list") ||
            !st.check(xkey.alloc(nw, s), "X list"))
            return failed();
        ak_xcount<<<grid_for(nw, 256), 256, 0, s>>>(d.w_idx, nw, xcnt.p);
        ak_xkeys<<<grid_for(nw, 256), 256, 0, s>>>(d.w_idx, nw, xkey.p);
        if (!scan_exclusive(xcnt.p, xcnt.p, K + 1, nullptr, s, st) ||
            !radix_sort(xkey, wown, nw, bits_for((uint64_t)K), s, st))
            return failed();
        d.x_off = (int *)xcnt.release();
        d.x_idx = (int *)wown.release();
    }
    // Stage 3c: leaves in sorted order, the leaf of every particle, tiles and their boxes.
    Buf<uint32_t> lflag, lscan;
    Buf<int> leaf_index, leaves;
    if (!st.check(lflag.alloc(n, s), "adaptive tree leaves") || !st.check(lscan.alloc(n, s), "adaptive tree leaves") ||
        !st.check(hipMemsetAsync(lflag.p, 0, n * sizeof(uint32_t), s), "adaptive tree leaves") ||
        !st.check(leaf_index.alloc(K, s), "adaptive tree leaves"))
        return failed();
    ak_leaf_marks<<<grid_for(K, 256), 256, 0, s>>>(d.cell, d.range, K, lflag.p);
    if (!scan_exclusive(lflag.p, lscan.p, n, nullptr, s, st)) return failed();
    if (!st.check(leaves.alloc(NL, s), "adaptive tree leaves") ||
        !alloc_to(d.leaf_start, (int64_t)NL + 1, s, st, "leaf offsets"))
        return failed();
    ak_leaf_index<<<grid_for(K, 256), 256, 0, s>>>(d.cell, d.range, K, lscan.p, leaf_index.p, leaves.p, d.leaf_start);
    ak_set<<<1, 1, 0, s>>>(d.leaf_start + NL, (int)n);
    ak_leaf_of<<<grid_for(n, 256), 256, 0, s>>>(lflag.p, lscan.p, leaves.p, n, d.leaf_of);
    Buf<uint32_t> ntile;
    if (!st.check(ntile.alloc((int64_t)NL + 1, s, true), "tiles")) return failed();
    ak_leaf_ntiles<<<grid_for((int64_t)NL + 1, 256), 256, 0, s>>>(leaves.p, d.range, (int)NL, ntile.p);
    if (!scan_exclusive(ntile.p, ntile.p, (int64_t)NL + 1, nullptr, s, st)) return failed();
    d.leaf_tile = (int *)ntile.release();  // NL + 1 entries, the last = the number of tiles

    // Stage 3d: the near-field plan, heaviest first.
    Buf<uint32_t> pcnt;
    Buf<unsigned long long> stats;
    uint32_t nwork = 0;
    if (!st.check(pcnt.alloc((int64_t)NL + 1, s), "near-field plan") ||
        !alloc_to(d.mask, K, s, st, "near-field mask") ||
        !st.check(hipMemsetAsync(d.mask, 0, (size_t)K * sizeof(uint16_t), s), "near-field mask") ||
        !st.check(stats.alloc(kStCount, s), "near-field plan") ||
        !st.check(hipMemsetAsync(stats.p, 0, kStCount * sizeof(unsigned long long), s), "near-field plan"))
        return failed();
    ak_plan<false><<<grid_for((int64_t)NL + 1, 256), 256, 0, s>>>(leaves.p, leaf_index.p, (int)NL, d.cell, d.range,
                                                                   coll.p, d.u_off, d.u_idx, t->dense_leaf, pcnt.p,
                                                                   nullptr, nullptr, nullptr, nullptr, d.mask,
                                                                   stats.p);
    unsigned long long hs[kStCount];
    uint32_t ntiles = 0;
    if (!scan_exclusive(pcnt.p, pcnt.p, (int64_t)NL + 1, nullptr, s, st) ||
        !st.check(hipMemcpyAsync(&nwork, pcnt.p + NL, sizeof nwork, hipMemcpyDeviceToHost, s), "near-field plan") ||
        !st.check(hipMemcpyAsync(&ntiles, d.leaf_tile + NL, sizeof ntiles, hipMemcpyDeviceToHost, s), "tiles") ||
        !read_back(hs, stats.p, sizeof hs, s, st))
        return failed();
    Buf<int> tile_leaf;
    if (!alloc_to(d.tile_start, K, s, st, "tiles") ||
        !st.check(hipMemsetAsync(d.tile_start, 0, (size_t)K * sizeof(int), s), "tiles") ||
        !st.check(tile_leaf.alloc(ntiles, s), "tiles") || !alloc_to(d.tile_box, ntiles, s, st, "tile boxes") ||
        !alloc_to(d.tile_box_leaf, ntiles, s, st, "tile boxes"))
        return failed();
    ak_tiles<<<grid_for(NL, 256), 256, 0, s>>>(leaves.p, d.leaf_tile, (int)NL, d.tile_start, tile_leaf.p);
    ak_tile_box<<<grid_for(ntiles, 256), 256, 0, s>>>(tile_leaf.p, leaves.p, d.leaf_tile, d.cell, d.range, d.xy,
                                                      ntiles, t->x0, t->y0, t->side, d.tile_box, d.tile_box_leaf);
    Buf<int4> work;
    Buf<uint64_t> cost;
    Buf<uint32_t> order;
    if (!st.check(work.alloc(nwork, s), "near-field plan") || !st.check(cost.alloc(nwork, s), "near-field plan") ||
        !st.check(order.alloc(nwork, s), "near-field plan"))
        return failed();
    ak_plan<true><<<grid_for((int64_t)NL + 1, 256), 256, 0, s>>>(leaves.p, leaf_index.p, (int)NL, d.cell, d.range,
                                                                  coll.p, d.u_off, d.u_idx, t->dense_leaf, nullptr,
                                                                  (const int *)pcnt.p, work.p, cost.p, order.p, nullptr,
                                                                  nullptr);
    if (!alloc_to(d.work, nwork, s, st, "near-field work")) return failed();
    if (!radix_sort(cost, order, nwork, 8, s, st)) return failed();
    ak_gather_work<<<grid_for(nwork, 256), 256, 0, s>>>(work.p, order.p, nwork, d.work);

    // Leaves and split cells of level >= 2, in cell order.
    const uint32_t ninner = (uint32_t)t->inner_off[L + 1];
    const uint32_t np2m = L >= 2 ? (uint32_t)(K - t->level_off[2]) - ninner : 0u;
    {
        Buf<uint32_t> fl, fi, pl, pi;
        if (!st.check(fl.alloc(K + 1, s), "adaptive tree build") || !st.check(fi.alloc(K + 1, s), "adaptive tree build") ||
            !st.check(pl.alloc(K + 1, s), "adaptive tree build") || !st.check(pi.alloc(K + 1, s), "adaptive tree build"))
            return failed();
        ak_cell_flags<<<grid_for(K + 1, 256), 256, 0, s>>>(d.cell, K, fl.p, fi.p);
        if (!scan_exclusive(fl.p, pl.p, K + 1, nullptr, s, st) || !scan_exclusive(fi.p, pi.p, K + 1, nullptr, s, st))
            return failed();
        if (!alloc_to(d.p2m_cells, np2m, s, st, "leaves with expansions") || !alloc_to(d.inner, ninner, s, st, "split cells"))
            return failed();
        ak_compact<<<grid_for(K, 256), 256, 0, s>>>(fl.p, pl.p, K, d.p2m_cells);
        ak_compact<<<grid_for(K, 256), 256, 0, s>>>(fi.p, pi.p, K, d.inner);
    }

    // Staging slots of the two-pass permutations between user and sorted order.
    t->stage_shift = stage_shift_of(n);
    if (!alloc_to(d.gpos1, n, s, st, "staging slots") || !alloc_to(d.gpos2, n, s, st, "staging slots") ||
        !alloc_to(d.st1, n, s, st, "staging array") || !build_staging(d.perm, n, s, st, t->stage_shift, d.gpos1, d.gpos2))
        return failed();

    int he = 0;
    if (!read_back(&he, werr.p, sizeof he, s, st) || !st.check(hipGetLastError(), "adaptive tree build")) return failed();
    if (he) {
        err = "adaptive tree: list walk deeper than the stack";
        return FMM_EDEVICE;
    }

    const int64_t sz[FMM_AT_COUNT] = {K, (int64_t)NL, (int64_t)nu, (int64_t)nv, (int64_t)nw, (int64_t)nw, deepest,
                                      (int64_t)hs[kStPairs]};
    std::copy(sz, sz + FMM_AT_COUNT, t->sizes);
    t->np2m = np2m;
    t->ntiles = ntiles;
    t->nwork = nwork;
    t->mutual_items = (int64_t)hs[kStMutualItems];
    t->mutual_pairs = (int64_t)hs[kStMutualPairs];
    t->target_units = (int64_t)hs[kStUnits];
    return FMM_OK;
}

int build_atree_adjoint_units(fmm_atree *t, hipStream_t s, std::string &err)
{
    Status st;
    BuildScope scope(s);
    const int64_t nt = t->ntiles;
    const int NL = (int)t->sizes[FMM_AT_LEAVES];
    Buf<int4> units;
    Buf<uint64_t> cost;
    Buf<uint32_t> order;
    int4 *out = nullptr;
    if (!st.check(units.alloc(nt, s), "adjoint units") || !st.check(cost.alloc(nt, s), "adjoint units") ||
        !st.check(order.alloc(nt, s), "adjoint units") || !alloc_to(out, nt, s, st, "adjoint units")) {
        err = st.msg;
        return st.code;
    }
    ak_adj_units<<<grid_for(NL, 256), 256, 0, s>>>(t->d.leaf_start, t->d.leaf_of, t->d.leaf_tile, NL, t->d.range,
                                                   t->d.u_off, t->d.u_idx, units.p, cost.p, order.p);
    const bool sorted = radix_sort(cost, order, nt, 8, s, st);
    if (sorted) ak_gather_work<<<grid_for(nt, 256), 256, 0, s>>>(units.p, order.p, nt, out);
    if (!sorted || !st.check(hipGetLastError(), "adjoint units") ||
        !st.check(hipStreamSynchronize(s), "adjoint units")) {
        build_free(out, (size_t)nt * sizeof(int4), s);
        err = st.msg;
        return st.code;
    }
    t->d.bwd_units = out;
    t->nbwd_units = nt;
    return FMM_OK;
}

// M2L plan of the MFMA path: segment key 4 (level - 2) + parity class and cell of every
// cell of level >= 2, and the counts per segment (count[0 .. 4 nlev - 1]).
__global__ __launch_bounds__(256) void ak_m2l_keys(const int4 *__restrict__ cell, int first, int ncl, int nseg,
                                                   uint64_t *__restrict__ key, uint32_t *__restrict__ val,
                                                   unsigned int *__restrict__ count)
{
    __shared__ unsigned int bc[64];
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (threadIdx.x < nseg) bc[threadIdx.x] = 0;
    __syncthreads();
    if (i < ncl) {
        const int4 c = cell[first + i];
        const int sg = 4 * (c.x - 2) + ((c.y & 1) | ((c.z & 1) << 1));
        key[i] = (uint64_t)sg;
        val[i] = (uint32_t)(first + i);
        atomicAdd(&bc[sg], 1u);
    }
    __syncthreads();
    if (threadIdx.x < nseg && bc[threadIdx.x]) atomicAdd(&count[threadIdx.x], bc[threadIdx.x]);
}

// Source cell of each interaction offset {dx, dy} of the cell's class (entries 28 q ..
// 28 q + 26 of the operator tables) from its V list; a V member of another level or at an
// offset outside the class's 27 counts into *bad.
// (vslot holds -1 before; eight lanes per cell.)
__global__ __launch_bounds__(256) void ak_vslot(const int4 *__restrict__ cell, int first, int ncl,
                                                const int *__restrict__ v_off, const int *__restrict__ v_idx,
                                                const int4 *__restrict__ entries, int *__restrict__ vslot,
                                                unsigned int *__restrict__ bad)
{
    __shared__ int place[4][49];  // of offset 7 (dx + 3) + dy + 3 among the class's 27, or -1
    for (int t = threadIdx.x; t < 4 * 49; t += 256) (&place[0][0])[t] = -1;
    __syncthreads();
    if (threadIdx.x < 4 * 27) {
        const int q = threadIdx.x / 27, j = threadIdx.x % 27;
        const int4 en = entries[28 * q + j];
        place[q][7 * (en.x + 3) + en.y + 3] = j;
    }
    __syncthreads();
    const int64_t i = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 3;
    if (i >= ncl) return;
    const int k = first + (int)i;
    const int4 c = cell[k];
    const int q = (c.y & 1) | ((c.z & 1) << 1);
    int *vs = vslot + i * 27;
    for (int e = v_off[k] + (threadIdx.x & 7); e < v_off[k + 1]; e += 8) {
        const int S = v_idx[e];
        const int4 cs = cell[S];
        const int dx = cs.y - c.y, dy = cs.z - c.z;
        const int slot = cs.x == c.x && abs(dx) <= 3 && abs(dy) <= 3 ? place[q][7 * (dx + 3) + dy + 3] : -1;
        if (slot < 0) atomicAdd(bad, 1u);
        else vs[slot] = S;
    }
}

int build_atree_m2l_plan(fmm_atree *t, const int4 *entries, hipStream_t s, std::string &err)
{
    Status st;
    const int deepest = (int)t->sizes[FMM_AT_DEEPEST];
    t->m2l_seg_off.assign(1, 0);
    if (deepest < 2) {
        t->m2l_plan = true;
        return FMM_OK;
    }
    const int first = t->level_off[2], ncl = t->level_off[deepest + 1] - first;
    const int nseg = 4 * (deepest - 1);  // <= 56
    BuildScope scope(s);
    Buf<uint64_t> key;
    Buf<uint32_t> val;
    Buf<unsigned int> cnt;
    int *targets = nullptr, *vslot = nullptr;
    auto failed = [&]() {
        build_free(targets, (size_t)std::max(ncl, 1) * sizeof(int), s);
        build_free(vslot, (size_t)std::max(ncl, 1) * 27 * sizeof(int), s);
        err = st.msg;
        return st.code;
    };
    if (!st.check(key.alloc(ncl, s), "M2L plan") || !st.check(val.alloc(ncl, s), "M2L plan") ||
        !st.check(cnt.alloc(nseg + 1, s), "M2L plan") ||
        !st.check(hipMemsetAsync(cnt.p, 0, (nseg + 1) * sizeof(unsigned int), s), "M2L plan") ||
        !alloc_to(targets, ncl, s, st, "M2L plan") || !alloc_to(vslot, 27 * (int64_t)ncl, s, st, "M2L plan"))
        return failed();
    ak_m2l_keys<<<grid_for(ncl, 256), 256, 0, s>>>(t->d.cell, first, ncl, nseg, key.p, val.p, cnt.p);
    if (!st.check(hipMemsetAsync(vslot, 0xff, 27 * (size_t)ncl * sizeof(int), s), "M2L plan")) return failed();
    ak_vslot<<<grid_for(8 * (int64_t)ncl, 256), 256, 0, s>>>(t->d.cell, first, ncl, t->d.v_off, t->d.v_idx, entries, vslot,
                                                cnt.p + nseg);
    // stable by segment: Morton order inside a class as inside a level
    if (!radix_sort(key, val, ncl, 6, s, st) ||
        !st.check(hipMemcpyAsync(targets, val.p, (size_t)ncl * sizeof(int), hipMemcpyDeviceToDevice, s), "M2L plan"))
        return failed();
    std::vector<unsigned int> hc((size_t)nseg + 1);
    if (!read_back(hc.data(), cnt.p, hc.size() * sizeof(unsigned int), s, st)) return failed();
    if (hc[nseg] != 0) {
        st.code = FMM_EDEVICE;
        st.msg = "M2L plan: " + std::to_string(hc[nseg]) + " V-list entries outside the interaction offsets";
        return failed();
    }
    t->m2l_seg_off.assign((size_t)nseg + 1, 0);
    for (int q = 0; q < nseg; ++q) t->m2l_seg_off[q + 1] = t->m2l_seg_off[q] + (int)hc[q];
    t->d.m2l_targets = targets;
    t->d.vslot = vslot;
    t->m2l_plan = true;
    return FMM_OK;
}

}  // namespace fmm
