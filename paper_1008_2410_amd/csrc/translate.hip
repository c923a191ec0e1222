// gfx950 kernels of the translations M2M, M2L and L2L (stages 5-7 of Fig. fmmStages of
// Knepley, arXiv:1008.2410), shared by the uniform and the adaptive tree.
//
// With radius-scaled coefficients every translation of one offset is the same 2p x 2p real
// operator (complex entries embedded with interleaved (re, im) rows and columns), so a tile
// of 16 (FP64) or 32 (FP32) targets of one parity class is a chain of small dense products
//   out(T) += sum_e row(source_e(T)) R_e
// on the matrix cores.  Absent sources read a zero row.
//
// A tree has few cells at most levels: the time of a chain of launches is the latency of a
// tile, not its arithmetic.  So the M2L of all levels, which needs only the multipoles, is
// one launch after the upward pass, and the downward pass is L2L alone, one operator per
// level, added to the locals the M2L wrote.  (With M2L + L2L fused per level, each level
// waited for the 28 gathered operands of the level above: 23-45 us a level whatever its
// size, and 77-135 us for the levels <= 3 in one workgroup.)
//
// Operand layouts (lane l):
//   FP64 16x16x4: A[row l%16][k l/16], B[k l/16][col l%16], D register r: [l/16 + 4r][l%16]
//   FP32 32x32x2: A[row l%32][k l/32], B[k l/32][col l%32], D register r:
//                 [8(r/4) + 4(l/32) + r%4][l%32]
// K is permuted so that a lane's steps are consecutive: step s of group g = l/16 (l/32) is
// k = KS g + s, so a lane reads KS contiguous values of its row.  The tables hold B as
// [slot][column block][16-byte vector of the lane's steps][lane], so that a wavefront reads
// an operator in whole cache lines (a lane's own steps in a row made each load touch four
// times the lines: 1024^2 lattice FP64, M2L of the finest level 96 us).
#include "translate.h"

#include <algorithm>

#include "device_common.h"

namespace fmm {
namespace {

typedef double doublex4 __attribute__((ext_vector_type(4)));
typedef float floatx16 __attribute__((ext_vector_type(16)));

__device__ __forceinline__ int find_seg(const TransArgs &a, int tile)
{
    int sg = 0;
    for (int k = 1; k < a.nseg; ++k)
        if (tile >= a.seg[k].tile0) sg = k;
    return sg;
}

// KS values of a row from k0 on; those from two_p on are not the row's (the reads stay inside
// the array's tail pad or the zero row) and enter the products as zero (in_row).  The
// selection waits until the value is used: at the load it would wait for memory there.
template <int KS>
__device__ __forceinline__ void load_row(double (&a)[KS], const double *row, int k0)
{
    const double2 *r = (const double2 *)(row + k0);
#pragma unroll
    for (int v = 0; v < KS / 2; ++v) {
        const double2 t = r[v];
        a[2 * v] = t.x;
        a[2 * v + 1] = t.y;
    }
}
template <typename T> __device__ __forceinline__ T in_row(T v, int k, int two_p) { return k < two_p ? v : (T)0; }

// This lane's steps of column block cb of an operator.
template <int KS, int NB>
__device__ __forceinline__ void load_op(double (&b)[KS], const double *tab, int slot, int cb, int lane)
{
    const double2 *t = (const double2 *)tab + ((size_t)slot * NB + cb) * (KS / 2) * 64 + lane;
#pragma unroll
    for (int v = 0; v < KS / 2; ++v) {
        const double2 u = t[v * 64];
        b[2 * v] = u.x;
        b[2 * v + 1] = u.y;
    }
}

// Blocks of 16 output columns.
template <int KS> constexpr int col_blocks() { return (4 * KS + 15) / 16; }

// ---------------------------------------------------------------------------------
// FP64.  A workgroup takes one tile of 16 RB targets; wavefront w has the column block
// w % NB and, of the tile's operators, every KG-th from w / NB on.  The KG partial sums
// meet in LDS, added in a fixed order; with SEQ one wavefront per column block makes them
// one after the other and adds them in that order, without LDS and to the same bits.
// Bound: the matrix cores (64 cycles per 16x16x4 product) where the tiles fill the chip,
// the latency of the gathered rows where they do not; hence the operands of the next
// operator are loaded ahead of the products of the current one, and few tiles are split
// further (KG).
// ---------------------------------------------------------------------------------
template <int KS, int RB, int KG, bool SEQ, Trans MODE, bool ADAPT>
__global__ __launch_bounds__(64 * col_blocks<KS>() * (SEQ ? 1 : KG)) void trans64_kernel(TransArgs a)
{
    constexpr int NB = col_blocks<KS>();
    constexpr int NE = MODE == Trans::M2L ? 27 : MODE == Trans::M2M ? 4 : 1;
    const int tile = xcd_block(kXcds);
    if (tile >= a.ntiles) return;  // the whole workgroup
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int cb = wave % NB, kg = wave / NB;
    const int row = lane & 15, kq = lane >> 4;
    const int two_p = 2 * a.p, k0 = KS * kq;
    const int sg = find_seg(a, tile);
    const TransSeg seg = a.seg[sg];
    const int q = sg & 3;
    const int base = (tile - seg.tile0) * 16 * RB;
    const int *tl = a.targets + seg.start;

    int tcell[RB], tx[RB], ty[RB];
#pragma unroll
    for (int b = 0; b < RB; ++b) {
        const int li = base + 16 * b + row;
        tcell[b] = li < seg.len ? tl[li] : -1;
        if constexpr (!ADAPT && MODE == Trans::M2L) {
            tx[b] = (int)morton_x((uint32_t)tcell[b]);
            ty[b] = (int)morton_y((uint32_t)tcell[b]);
        }
    }
    const int64_t here = ADAPT ? 0 : level_base(seg.level) - a.out_off;
    const int64_t from =
        ADAPT ? 0 : level_base(seg.level + (MODE == Trans::M2M ? 1 : MODE == Trans::L2L ? -1 : 0)) - a.src_off;
    const bool second = blockIdx.y != 0;
    const double *src = (const double *)(second ? a.src2 : a.src);
    double *out = (double *)(second ? a.out2 : a.out);
    const double *par = (const double *)(second ? a.par2 : a.par);

    // the source row of target block b for operator e, or the zero row: selected, not
    // branched over, so that the loads of the next operator stay in flight
    auto source = [&](int b, int e, int4 en) -> const double * {
        const int64_t c = max(tcell[b], 0);
        bool ok = tcell[b] >= 0 && e >= 0;
        e = max(e, 0);
        int64_t S;
        const double *rows = src;
        if constexpr (MODE == Trans::M2L && !ADAPT) {
            const uint32_t nside = 1u << seg.level;
            const uint32_t sx = (uint32_t)(tx[b] + en.x), sy = (uint32_t)(ty[b] + en.y);
            const bool l2l = e == 27;  // wavefront-uniform
            ok = ok && (l2l || (sx < nside && sy < nside));
            S = l2l ? level_base(seg.level - 1) - a.par_off + (c >> 2) : from + morton_encode(sx, sy);
            rows = l2l ? par : src;
        } else if constexpr (MODE == Trans::M2M && !ADAPT) {
            S = from + 4 * c + e;
        } else if constexpr (MODE == Trans::L2L && !ADAPT) {
            S = from + (c >> 2);
        } else if constexpr (MODE == Trans::M2L) {
            S = a.vslot[(ok ? c - a.first : 0) * 27 + e];
            ok = ok && S >= 0;
        } else if constexpr (MODE == Trans::M2M) {
            S = ((const int *)(a.child + c))[e];
            ok = ok && S >= 0;
        } else {
            S = a.parent[c];
            ok = ok && S >= 0;
        }
        return ok ? rows + S * two_p : a.zero;
    };
    const int e0 = MODE == Trans::M2L ? 28 * q : MODE == Trans::M2M ? 112 : 28 * q + 27;

    // operators this wavefront applies, as a bit mask (adaptive M2L: those some target uses)
    uint32_t used = (1u << NE) - 1u;
    if (MODE == Trans::M2L && !ADAPT && a.par) used |= 1u << 27;
    if constexpr (ADAPT && MODE == Trans::M2L) {
        used = 0;
#pragma unroll
        for (int e = 0; e < NE; ++e) {
            bool any = false;
#pragma unroll
            for (int b = 0; b < RB; ++b)
                any = any || (tcell[b] >= 0 && a.vslot[(int64_t)(tcell[b] - a.first) * 27 + e] >= 0);
            if (__any(any)) used |= 1u << e;
        }
    }
    // every KG-th of them, from number g on
    auto share = [](uint32_t all, int g) {
        uint32_t mine = 0;
        for (int k = 0; all; ++k) {
            const uint32_t low = all & -all;
            if (k % KG == g) mine |= low;
            all ^= low;
        }
        return mine;
    };
    used = (uint32_t)__builtin_amdgcn_readfirstlane((int)used);

    doublex4 acc[RB];
#pragma unroll
    for (int b = 0; b < RB; ++b)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[b][r] = 0.0;
    const int col = 16 * cb + row;
    if ((MODE == Trans::L2L || (ADAPT && MODE == Trans::M2L)) && kg == 0) {
#pragma unroll
        for (int b = 0; b < RB; ++b)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int o = base + 16 * b + kq + 4 * r;
                if (o < seg.len && col < two_p) {
                    const int k = tl[o];
                    // L2L adds to the M2L sums; the adaptive M2L to the P2L sums, where there are any
                    if (MODE == Trans::L2L || a.x_off[k] < a.x_off[k + 1]) acc[b][r] = out[(here + k) * two_p + col];
                }
            }
    }

    const double *tab = (const double *)a.tab;
    double av[2][RB][KS], bv[2][KS];
    auto fetch = [&](int slot, int e) {  // e < 0: none (zero rows)
        const int4 en = a.entries[e0 + max(e, 0)];
        load_op<KS, NB>(bv[slot], tab, en.z, cb, lane);
#pragma unroll
        for (int b = 0; b < RB; ++b) load_row<KS>(av[slot][b], source(b, e, en), k0);
        __builtin_amdgcn_sched_barrier(0);  // the loads go out before the products that follow
    };
    auto products = [&](int slot) {
#pragma unroll
        for (int s = 0; s < KS; ++s)
#pragma unroll
            for (int b = 0; b < RB; ++b)
                acc[b] = __builtin_amdgcn_mfma_f64_16x16x4f64(in_row(av[slot][b][s], k0 + s, two_p), bv[slot][s], acc[b],
                                                              0, 0, 0);
    };
    // the operators of m (wavefront-uniform) in order, the next one's operands loaded ahead of
    // the products of the current one, without a branch between them (a load whose use is
    // behind a branch moves down to it)
    auto apply = [&](uint32_t m) {
        auto next = [&m]() {
            const int e = m ? __builtin_ctz(m) : -1;
            m &= m - 1;
            return e;
        };
        if constexpr (NE == 1) {
            fetch(0, 0);
            products(0);
        } else {
            int e = next();
            if (e < 0) return;
            fetch(0, e);
            do {
                fetch(1, next());
                products(0);
                e = next();
                fetch(0, e);
                products(1);
            } while (e >= 0);
        }
    };
    if constexpr (KG == 1) {
        apply(used);
    } else if constexpr (SEQ) {
        doublex4 sum[RB];
        for (int g = 0; g < KG; ++g) {
            apply(share(used, g));
#pragma unroll
            for (int b = 0; b < RB; ++b)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    sum[b][r] = g == 0 ? acc[b][r] : sum[b][r] + acc[b][r];
                    acc[b][r] = 0.0;
                }
        }
#pragma unroll
        for (int b = 0; b < RB; ++b) acc[b] = sum[b];
    } else {
        apply(share(used, kg));
    }

    if constexpr (KG > 1 && !SEQ) {
        __shared__ double part[KG - 1][NB][RB][4][64];
        if (kg > 0)
#pragma unroll
            for (int b = 0; b < RB; ++b)
#pragma unroll
                for (int r = 0; r < 4; ++r) part[kg - 1][cb][b][r][lane] = acc[b][r];
        __syncthreads();
        if (kg > 0) return;
#pragma unroll
        for (int g = 0; g < KG - 1; ++g)
#pragma unroll
            for (int b = 0; b < RB; ++b)
#pragma unroll
                for (int r = 0; r < 4; ++r) acc[b][r] += part[g][cb][b][r][lane];
    }
#pragma unroll
    for (int b = 0; b < RB; ++b)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int o = base + 16 * b + kq + 4 * r;
            if (o < seg.len && col < two_p) out[(here + tl[o]) * two_p + col] = acc[b][r];
        }
}

// ---------------------------------------------------------------------------------
// The coarse end of the upward and downward passes: one workgroup per cell of level `base`
// takes its subtree's next three levels in sequence, every cell of them (rows of empty
// cells stay zero going up, and are not read going down).  A level is at most one 16-row
// tile of parents going up (a wavefront per column block) and one per parity class going
// down (a wavefront per class), so three levels cost three tile latencies and one launch.
// ---------------------------------------------------------------------------------
template <int KS>
__global__ __launch_bounds__(64 * col_blocks<KS>()) void subtree_up_kernel(SubtreeArgs a)
{
    constexpr int NB = col_blocks<KS>();
    double *const rows = blockIdx.y ? a.rows2 : a.rows;
    const int cell0 = blockIdx.x;
    if (a.counts[level_base(a.base) + cell0] == 0) return;
    const int lane = threadIdx.x & 63, cb = threadIdx.x >> 6;
    const int row = lane & 15, kq = lane >> 4;
    const int two_p = 2 * a.p, k0 = KS * kq, col = 16 * cb + row;
    for (int l = min(a.deepest - 1, a.base + 2); l >= a.base; --l) {
        const int n = 1 << (2 * (l - a.base));
        const double *child = rows + (level_base(l + 1) + 4 * ((int64_t)cell0 * n + min(row, n - 1))) * two_p;
        double av[4][KS], bv[4][KS];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            load_row<KS>(av[e], child + e * two_p, k0);
            load_op<KS, NB>(bv[e], a.tab, 53 + e, cb, lane);
        }
        doublex4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int s = 0; s < KS; ++s)
                acc = __builtin_amdgcn_mfma_f64_16x16x4f64(in_row(av[e][s], k0 + s, two_p), bv[e][s], acc, 0, 0, 0);
        double *out = rows + (level_base(l) + (int64_t)cell0 * n) * two_p;
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (kq + 4 * r < n && col < two_p) out[(kq + 4 * r) * two_p + col] = acc[r];
        __syncthreads();  // the next level reads these rows
    }
}

template <int KS> __global__ __launch_bounds__(256) void subtree_down_kernel(SubtreeArgs a)
{
    constexpr int NB = col_blocks<KS>();
    double *const rows = blockIdx.y ? a.rows2 : a.rows;
    const int cell0 = blockIdx.x;
    if (a.counts[level_base(a.base) + cell0] == 0) return;
    const int lane = threadIdx.x & 63, q = threadIdx.x >> 6;  // wavefront: parity class of the targets
    const int row = lane & 15, kq = lane >> 4;
    const int two_p = 2 * a.p, k0 = KS * kq;
    double bv[NB][KS];  // the class's operator, the same at every level
#pragma unroll
    for (int c = 0; c < NB; ++c)
        load_op<KS, NB>(bv[c], a.tab, 49 + q, c, lane);
    for (int l = a.base + 1; l <= min(a.deepest, a.base + 3); ++l) {
        const int n = 1 << (2 * (l - a.base - 1));  // parents in the subtree, one target each per class
        const double *par = rows + (level_base(l - 1) + (int64_t)cell0 * n) * two_p;
        double *out = rows + (level_base(l) + 4 * (int64_t)cell0 * n + q) * two_p;  // target of parent k: row 4 k
        double av[KS];
        load_row<KS>(av, par + (int64_t)min(row, n - 1) * two_p, k0);
        doublex4 acc[NB];
#pragma unroll
        for (int c = 0; c < NB; ++c)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int o = kq + 4 * r;
                acc[c][r] = o < n && 16 * c + row < two_p ? out[(int64_t)4 * o * two_p + 16 * c + row] : 0.0;
            }
#pragma unroll
        for (int s = 0; s < KS; ++s)
#pragma unroll
            for (int c = 0; c < NB; ++c)
                acc[c] = __builtin_amdgcn_mfma_f64_16x16x4f64(in_row(av[s], k0 + s, two_p), bv[c][s], acc[c], 0, 0, 0);
#pragma unroll
        for (int c = 0; c < NB; ++c)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int o = kq + 4 * r;
                if (o < n && 16 * c + row < two_p) out[(int64_t)4 * o * two_p + 16 * c + row] = acc[c][r];
            }
        __syncthreads();  // the next level reads these rows
    }
}

// ---------------------------------------------------------------------------------
// The same for the adaptive tree: one workgroup per split cell of level `base`, its descendants
// found through the child indices.  A row of the tile of level base + 1 (+ 2) is a place in the
// subtree, quadrant by quadrant; places without a cell read the zero row and are not written.
// A level of its own cost a launch of 5 us whatever it held (150001 clustered particles: 60
// launches of a gradient's 700 us), and one launch of three levels costs 8.
// ---------------------------------------------------------------------------------
__device__ __forceinline__ int pick(int4 c, int q) { return q == 0 ? c.x : q == 1 ? c.y : q == 2 ? c.z : c.w; }

// Lane row r of a wavefront: its cell at level base + d (d = 0, 1, 2; -1: none) and that cell's
// children.
struct SubtreePlaces {
    int id[3];
    int4 ch[3];
    __device__ __forceinline__ SubtreePlaces(const SubtreeArgs &a, int cell0, int row)
    {
        const int4 none = make_int4(-1, -1, -1, -1);
        const int4 c0 = a.child[cell0];
        id[0] = row == 0 ? cell0 : -1;
        ch[0] = row == 0 ? c0 : none;
        id[1] = row < 4 ? pick(c0, row & 3) : -1;
        const int i1 = pick(c0, row >> 2);
        const int4 g = a.child[max(i1, 0)];
        ch[1] = a.child[max(id[1], 0)];
        if (id[1] < 0) ch[1] = none;
        id[2] = i1 >= 0 ? pick(g, row & 3) : -1;
        ch[2] = a.child[max(id[2], 0)];
        if (id[2] < 0) ch[2] = none;
    }
};

template <int KS>
__global__ __launch_bounds__(64 * col_blocks<KS>()) void subtree_up_adaptive_kernel(SubtreeArgs a)
{
    constexpr int NB = col_blocks<KS>();
    double *const rows = blockIdx.y ? a.rows2 : a.rows;
    const int lane = threadIdx.x & 63, cb = threadIdx.x >> 6;
    const int row = lane & 15, kq = lane >> 4;
    const int two_p = 2 * a.p, k0 = KS * kq, col = 16 * cb + row;
    double bv[4][KS];
#pragma unroll
    for (int e = 0; e < 4; ++e) load_op<KS, NB>(bv[e], a.tab, 53 + e, cb, lane);
    const SubtreePlaces pl(a, a.cells[blockIdx.x], row);
#pragma unroll
    for (int d = 2; d >= 0; --d) {
        if (a.base + d > a.deepest - 1) continue;  // (no level below)
        const int4 ch = pl.ch[d];
        // a cell without children is a leaf, whose row the particles gave
        const int target = max(max(ch.x, ch.y), max(ch.z, ch.w)) >= 0 ? pl.id[d] : -1;
        if (__any(target >= 0)) {
            double av[4][KS];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int S = pick(ch, e);
                load_row<KS>(av[e], S >= 0 ? rows + (int64_t)S * two_p : a.zero, k0);
            }
            doublex4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int s = 0; s < KS; ++s)
                    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(in_row(av[e][s], k0 + s, two_p), bv[e][s], acc, 0, 0, 0);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int t = __shfl(target, kq + 4 * r);
                if (t >= 0 && col < two_p) rows[(int64_t)t * two_p + col] = acc[r];
            }
        }
        __syncthreads();  // the next level reads these rows
    }
}

template <int KS> __global__ __launch_bounds__(256) void subtree_down_adaptive_kernel(SubtreeArgs a)
{
    constexpr int NB = col_blocks<KS>();
    double *const rows = blockIdx.y ? a.rows2 : a.rows;
    const int lane = threadIdx.x & 63, q = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int row = lane & 15, kq = lane >> 4;
    const int two_p = 2 * a.p, k0 = KS * kq;
    double bv[NB][KS];  // the class's operator, the same at every level
#pragma unroll
    for (int c = 0; c < NB; ++c) load_op<KS, NB>(bv[c], a.tab, 49 + q, c, lane);
    const SubtreePlaces pl(a, a.cells[blockIdx.x], row);
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        if (a.base + d > a.deepest - 1) continue;  // (no level below)
        const int target = pick(pl.ch[d], q);
        if (__any(target >= 0)) {
            double av[KS];
            load_row<KS>(av, target >= 0 ? rows + (int64_t)pl.id[d] * two_p : a.zero, k0);
            int to[4];
            doublex4 acc[NB];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                to[r] = __shfl(target, kq + 4 * r);
#pragma unroll
                for (int c = 0; c < NB; ++c)
                    acc[c][r] = to[r] >= 0 && 16 * c + row < two_p ? rows[(int64_t)to[r] * two_p + 16 * c + row] : 0.0;
            }
#pragma unroll
            for (int s = 0; s < KS; ++s)
#pragma unroll
                for (int c = 0; c < NB; ++c)
                    acc[c] = __builtin_amdgcn_mfma_f64_16x16x4f64(in_row(av[s], k0 + s, two_p), bv[c][s], acc[c], 0, 0, 0);
#pragma unroll
            for (int c = 0; c < NB; ++c)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (to[r] >= 0 && 16 * c + row < two_p) rows[(int64_t)to[r] * two_p + 16 * c + row] = acc[c][r];
        }
        __syncthreads();  // the next level reads these rows
    }
}

// ---------------------------------------------------------------------------------
// FP32 (the fine levels of the mixed form): one wavefront per tile of 32 targets and block
// of 32 columns, the next operator's operands loaded ahead of the current one's products.
// ---------------------------------------------------------------------------------
template <int KF>
__device__ __forceinline__ void load_row32(float (&a)[KF], const float *row)
{
#pragma unroll
    for (int s = 0; s < KF; ++s) a[s] = row[s];
}
template <int KF>
__device__ __forceinline__ void load_row32(float (&a)[KF], const double *row)
{
#pragma unroll
    for (int s = 0; s < KF; ++s) a[s] = (float)row[s];
}

template <int KF> constexpr int col_blocks32() { return KF <= 16 ? 1 : 2; }

template <int KF, Trans MODE, typename TSrc, typename TOut>
__global__ __launch_bounds__(256, KF <= 16 ? 4 : 2) void trans32_kernel(TransArgs a)
{
    constexpr int NB = col_blocks32<KF>();
    // M2L: the 28th is the L2L (with par), else nothing (zero rows)
    constexpr int NE = MODE == Trans::M2L ? 28 : MODE == Trans::M2M ? 4 : 1;
    const int lane = threadIdx.x & 63;
    const int id = xcd_block(kXcds) * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int tile = id / NB, cb = id % NB;
    if (tile >= a.ntiles) return;  // whole wavefronts; no barriers below
    const int row = lane & 31, kh = lane >> 5;
    const int two_p = 2 * a.p, k0 = KF * kh;
    const int sg = find_seg(a, tile);
    const TransSeg seg = a.seg[sg];
    const int q = sg & 3;
    const int base = (tile - seg.tile0) * 32;
    const int *tl = a.targets + seg.start;
    const int li = base + row;
    const int tcell = li < seg.len ? tl[li] : -1;
    const int tx = (int)morton_x((uint32_t)tcell), ty = (int)morton_y((uint32_t)tcell);
    const int64_t here = level_base(seg.level) - a.out_off;
    const int64_t from = level_base(seg.level + (MODE == Trans::M2M ? 1 : MODE == Trans::L2L ? -1 : 0)) - a.src_off;
    const bool second = blockIdx.y != 0;
    const TSrc *src = (const TSrc *)(second ? a.src2 : a.src);
    TOut *out = (TOut *)(second ? a.out2 : a.out);
    const float *par = (const float *)(second ? a.par2 : a.par);
    const float *tab = (const float *)a.tab;
    const int e0 = MODE == Trans::M2L ? 28 * q : MODE == Trans::M2M ? 112 : 28 * q + 27;
    const int col = 32 * cb + row;

    floatx16 acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
    if constexpr (MODE == Trans::L2L) {  // added to the M2L sums
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int cell = __shfl(tcell, 8 * (r >> 2) + 4 * kh + (r & 3));
            if (cell >= 0 && col < two_p) acc[r] = (float)out[(here + cell) * two_p + col];
        }
    }
    float av[2][KF], bv[2][KF];
    auto fetch = [&](int slot, int e) {
        const int4 en = a.entries[e0 + e];
        const float4 *b = (const float4 *)tab + ((size_t)en.z * NB + cb) * (KF / 4) * 64 + lane;
#pragma unroll
        for (int v = 0; v < KF / 4; ++v) {
            const float4 t = b[v * 64];
            bv[slot][4 * v] = t.x;
            bv[slot][4 * v + 1] = t.y;
            bv[slot][4 * v + 2] = t.z;
            bv[slot][4 * v + 3] = t.w;
        }
        // selected, not branched over (see trans64_kernel)
        const int64_t c = max(tcell, 0);
        if constexpr (MODE == Trans::M2L) {
            const uint32_t nside = 1u << seg.level;
            const uint32_t sx = (uint32_t)(tx + en.x), sy = (uint32_t)(ty + en.y);
            const int64_t S = from + morton_encode(sx, sy);
            const bool l2l = e == 27 && a.par;  // wavefront-uniform
            const int64_t P = level_base(seg.level - 1) - a.par_off + (c >> 2);
            const float *r = (l2l ? par : (const float *)src) + (l2l ? P : S) * two_p;
            const bool ok = tcell >= 0 && (l2l || (e < 27 && sx < nside && sy < nside));
            r = ok ? r : (const float *)a.zero;
            load_row32<KF>(av[slot], r + k0);
        } else {
            const int64_t S = from + (MODE == Trans::M2M ? 4 * c + e : c >> 2);
            load_row32<KF>(av[slot], (tcell >= 0 ? src + S * two_p : (const TSrc *)a.zero) + k0);
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    auto products = [&](int slot) {
#pragma unroll
        for (int s = 0; s < KF; ++s)
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(in_row(av[slot][s], k0 + s, two_p), bv[slot][s], acc, 0, 0, 0);
    };
    // the next operator's operands ahead of the current one's products (see trans64_kernel)
    fetch(0, 0);
    if constexpr (NE == 1) {
        products(0);
    } else {
        for (int e = 0; e < NE; e += 2) {
            fetch(1, e + 1);
            products(0);
            fetch(0, min(e + 2, NE - 1));
            products(1);
        }
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int cell = __shfl(tcell, 8 * (r >> 2) + 4 * kh + (r & 3));
        if (cell >= 0 && col < two_p) out[(here + cell) * two_p + col] = (TOut)acc[r];
    }
}

// Number the tiles of the segments (of `rows` targets each).
void number_tiles(TransArgs &a, int rows)
{
    a.ntiles = 0;
    for (int k = 0; k < a.nseg; ++k) {
        a.seg[k].tile0 = a.ntiles;
        a.ntiles += (a.seg[k].len + rows - 1) / rows;
    }
}

template <int KS, int RB, int KG, Trans MODE, bool ADAPT, bool SEQ = false> void go64(TransArgs &a, hipStream_t s)
{
    number_tiles(a, 16 * RB);
    if (a.ntiles == 0) return;
    trans64_kernel<KS, RB, KG, SEQ, MODE, ADAPT>
        <<<dim3(xcd_grid(a.ntiles, 1, kXcds), a.out2 ? 2 : 1), 64 * col_blocks<KS>() * (SEQ ? 1 : KG), 0, s>>>(a);
}

// KG partial sums side by side, or one after the other where the LDS is held.
template <int KS, int KG, bool ADAPT> void split64(TransArgs &a, hipStream_t s)
{
    if (a.no_lds) go64<KS, 1, KG, Trans::M2L, ADAPT, true>(a, s);
    else go64<KS, 1, KG, Trans::M2L, ADAPT>(a, s);
}

// M2L: split the operators over more wavefronts while the tiles leave the chip's 1024 SIMDs
// idle; once they fill it, tiles of 32 targets (up to 16 terms: the operands of two row
// blocks fit the registers twice) read each operator half as often.  The split meets in
// LDS, so beside a near field that holds the LDS it would wait for workgroups to retire
// (2^24 patches: 3.4 ms for the 88 tiles of levels 2..5).
template <int KS, bool ADAPT> void m2l64(TransArgs &a, hipStream_t s)
{
    constexpr int NB = col_blocks<KS>();
    number_tiles(a, 16);
    const int waves = a.ntiles * NB;
    if constexpr (KS <= 8) {
        if (waves <= 1024) split64<KS, 4, ADAPT>(a, s);
        else if (waves <= 4096) go64<KS, 1, 1, Trans::M2L, ADAPT>(a, s);
        else go64<KS, 2, 1, Trans::M2L, ADAPT>(a, s);
    } else {
        if (waves <= 1024) split64<KS, 2, ADAPT>(a, s);
        else go64<KS, 1, 1, Trans::M2L, ADAPT>(a, s);
    }
}

template <int KS> void trans64(TransArgs &a, Trans mode, bool adaptive, hipStream_t s)
{
    if (mode == Trans::M2L) adaptive ? m2l64<KS, true>(a, s) : m2l64<KS, false>(a, s);
    else if (mode == Trans::M2M)
        adaptive ? go64<KS, 1, 1, Trans::M2M, true>(a, s) : go64<KS, 1, 1, Trans::M2M, false>(a, s);
    else adaptive ? go64<KS, 1, 1, Trans::L2L, true>(a, s) : go64<KS, 1, 1, Trans::L2L, false>(a, s);
}

template <int KF, Trans MODE, typename TSrc, typename TOut> void go32(TransArgs &a, hipStream_t s)
{
    trans32_kernel<KF, MODE, TSrc, TOut><<<dim3(xcd_grid((int64_t)a.ntiles * col_blocks32<KF>(), 4, kXcds), a.out2 ? 2 : 1), 256, 0, s>>>(a);
}

template <int KF> void trans32(TransArgs &a, Trans mode, bool src_double, bool out_double, hipStream_t s)
{
    if (mode == Trans::M2L) go32<KF, Trans::M2L, float, float>(a, s);
    else if (mode == Trans::M2M)
        out_double ? go32<KF, Trans::M2M, float, double>(a, s) : go32<KF, Trans::M2M, float, float>(a, s);
    else src_double ? go32<KF, Trans::L2L, double, float>(a, s) : go32<KF, Trans::L2L, float, float>(a, s);
}

template <int KS> void subtree(const SubtreeArgs &a, bool up, hipStream_t s)
{
    if (a.cells) {
        const dim3 g((unsigned)a.ncells, a.rows2 ? 2 : 1);
        if (up) subtree_up_adaptive_kernel<KS><<<g, 64 * col_blocks<KS>(), 0, s>>>(a);
        else subtree_down_adaptive_kernel<KS><<<g, 256, 0, s>>>(a);
        return;
    }
    const dim3 g(1u << (2 * a.base), a.rows2 ? 2 : 1);
    if (up) subtree_up_kernel<KS><<<g, 64 * col_blocks<KS>(), 0, s>>>(a);
    else subtree_down_kernel<KS><<<g, 256, 0, s>>>(a);
}

}  // namespace

void launch_trans64(TransArgs a, Trans mode, bool adaptive, hipStream_t s)
{
    switch (trans_ks(a.p)) {
    case 4: trans64<4>(a, mode, adaptive, s); break;
    case 6: trans64<6>(a, mode, adaptive, s); break;
    case 8: trans64<8>(a, mode, adaptive, s); break;
    case 12: trans64<12>(a, mode, adaptive, s); break;
    default: trans64<16>(a, mode, adaptive, s); break;
    }
}

void launch_trans32(TransArgs a, Trans mode, bool src_double, bool out_double, hipStream_t s)
{
    number_tiles(a, 32);
    if (a.ntiles == 0) return;
    switch (trans_kf(a.p)) {
    case 8: trans32<8>(a, mode, src_double, out_double, s); break;
    case 12: trans32<12>(a, mode, src_double, out_double, s); break;
    case 16: trans32<16>(a, mode, src_double, out_double, s); break;
    case 24: trans32<24>(a, mode, src_double, out_double, s); break;
    default: trans32<32>(a, mode, src_double, out_double, s); break;
    }
}

void launch_subtree(const SubtreeArgs &a, bool up, hipStream_t s)
{
    switch (trans_ks(a.p)) {
    case 4: subtree<4>(a, up, s); break;
    case 6: subtree<6>(a, up, s); break;
    case 8: subtree<8>(a, up, s); break;
    case 12: subtree<12>(a, up, s); break;
    default: subtree<16>(a, up, s); break;
    }
}

}  // namespace fmm
