// C ABI of the gfx950 FMM library (include/fmm2d.h): argument checks, the trees' lifetime
// (built by tree_build.hip or host_tree.cpp), workspace management and the two-stream
// schedule of stages 4-10.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <functional>
#include <new>
#include <numeric>
#include <string>
#include <vector>

#include "../../include/fmm2d.h"
#include "api_common.h"
#include "build_prims.h"
#include "fmm_internal.h"

using namespace fmm;

namespace {

thread_local std::string g_last_error;

// RAII guard for "one host thread per handle".
struct BusyGuard {
    fmm_tree *t;
    bool ok;
    explicit BusyGuard(fmm_tree *tree) : t(tree), ok(tree->busy.exchange(1) == 0) {}
    ~BusyGuard() { release(); }
    void release()
    {
        if (ok) t->busy.store(0);
        ok = false;
    }
};

// The workspace's blocks go to the library's cache; callers have finished the device work
// that used it (destroy) or synchronised (reallocation).
void free_workspace(Workspace &ws)
{
    for (void *p : {ws.gam, (void *)ws.stage, (void *)ws.near, (void *)ws.mp_d, (void *)ws.lo_d, (void *)ws.mp_f,
                    (void *)ws.lo_f, (void *)ws.adj, (void *)ws.mp2_d, (void *)ws.lo2_d, (void *)ws.mp2_f,
                    (void *)ws.lo2_f, (void *)ws.rec2, ws.sums, ws.phi_slots, (void *)ws.range})
        block_free(p);
    ws = Workspace{};
}

// The tree's device arrays (not its workspace, stream or events), freed in the order of
// stream fs; the caller has finished the work that used them.  Arrays of the device build
// come from the stream-ordered pool (those of fixed size in one slab), those of the host
// build from hipMalloc; the near-field plan and the leaf-unit coordinates are always pooled.
void release_tree_arrays(fmm_tree *t, hipStream_t fs)
{
    auto release = [fs](auto *&p, bool pooled) {
        if (!p) return;
        if (pooled) hipFreeAsync((void *)p, fs);
        else hipFree((void *)p);
        p = nullptr;
    };
    if (t->slab) {
        release(t->slab, true);
        t->d_perm = t->d_gpos1 = t->d_gpos2 = t->d_leaf_of = t->d_leaf_start = t->d_counts = t->d_tile_start = nullptr;
        t->d_st1 = nullptr;
        t->d_xy = nullptr;
        t->d_leaf_mask = nullptr;
    }
    release(t->d_perm, false);
    release(t->d_gpos1, false);
    release(t->d_gpos2, false);
    release(t->d_st1, false);
    release(t->d_leaf_of, false);
    release(t->d_xy, false);
    release(t->d_leaf_start, false);
    release(t->d_counts, false);
    release(t->d_tile_start, false);
    release(t->d_lists, t->pooled);
    release(t->d_units, t->pooled);
    release(t->d_tile_box, t->pooled);
    release(t->d_near_work, true);
    release(t->d_split, true);
    release(t->d_parts, true);
    release(t->d_part_sums, true);
    t->cap_split = t->cap_parts = t->cap_part_sums = 0;
    release(t->d_leaf_mask, true);
    t->cap_lists = t->cap_units = t->cap_tile_box = t->cap_near_work = 0;
    for (int k = 0; k < 2; ++k) {
        release(t->pos_buf[k], true);
        t->d_pos[k] = nullptr;
    }
}

// The arrays of a device-built tree pass to the tree rebuilt from it (same n and depth);
// the caller has finished the work that used them.
void take_over_arrays(fmm_tree *t, fmm_tree *from)
{
    auto take = [](auto &to, auto &of) {
        to = of;
        of = {};
    };
    take(t->slab, from->slab);
    take(t->d_perm, from->d_perm);
    take(t->d_gpos1, from->d_gpos1);
    take(t->d_gpos2, from->d_gpos2);
    take(t->d_st1, from->d_st1);
    take(t->d_leaf_of, from->d_leaf_of);
    take(t->d_xy, from->d_xy);
    take(t->d_leaf_start, from->d_leaf_start);
    take(t->d_counts, from->d_counts);
    take(t->d_tile_start, from->d_tile_start);
    take(t->d_leaf_mask, from->d_leaf_mask);
    take(t->d_lists, from->d_lists);
    take(t->d_units, from->d_units);
    take(t->d_tile_box, from->d_tile_box);
    take(t->d_near_work, from->d_near_work);
    take(t->cap_lists, from->cap_lists);
    take(t->cap_units, from->cap_units);
    take(t->cap_tile_box, from->cap_tile_box);
    take(t->cap_near_work, from->cap_near_work);
    take(t->d_split, from->d_split);
    take(t->d_parts, from->d_parts);
    take(t->d_part_sums, from->d_part_sums);
    take(t->cap_split, from->cap_split);
    take(t->cap_parts, from->cap_parts);
    take(t->cap_part_sums, from->cap_part_sums);
    for (int k = 0; k < 2; ++k) {
        take(t->pos_buf[k], from->pos_buf[k]);
        from->d_pos[k] = nullptr;
    }
}

void free_tree(fmm_tree *t)
{
    hipStream_t fs = t->aux.stream;  // the caller has finished the work on the tree
    release_tree_arrays(t, fs);
    hipFree(t->d_flag);
    if (t->wsp.use_count() == 1) free_workspace(*t->wsp);
    if (fs) hipStreamSynchronize(fs);  // the frees are in its order
    bound_idle(t->device);
    side_stream_give(t->device, t->aux);
    for (auto &evs : t->pending_timing)
        for (auto e : evs) hipEventDestroy(e);
    delete t;
}

// The mutual form is used when its plan has items; else the target-centric units alone.
bool use_mutual(const fmm_tree *t) { return t->near_mutual && t->nmut > 0; }

// Output bytes per particle by which the adjoint's route is chosen (dl_dgamma, and two parts of dl_dxy).
constexpr int64_t kForceRow = 40;

// Last FP64 level: every level in FP64 precision; in the mixed form the coarse levels, and
// always levels 2..5, whose few cells cost nothing in FP64 (their passes run in one launch).
constexpr int kMinSplit = 5;
int split_level(const fmm_tree *t, int precision)
{
    return precision == FMM_FP64 ? t->depth : std::min(std::max(t->lc, kMinSplit), t->depth);
}

// A workspace last used by another tree (a rebuild's hand-over, or a tree sharing it):
// multipoles of cells that are empty in this tree must read as zero (the M2L kernels
// read them unconditionally), so the multipole arrays are cleared, by a kernel: the call
// may be captured, and memset nodes of a graph are not relied on.  Locals and
// per-particle arrays are written in full by every call before they are read.
int clear_multipoles(const fmm_tree *t, hipStream_t s)
{
    const Workspace &ws = *t->wsp;
    if (!ws.gam || t->depth < 2) return FMM_OK;
    const int64_t cells_d = level_base(std::min(ws.split, t->depth) + 1);
    const int64_t cells_f = level_base(t->depth + 1) - cells_d;
    const size_t bd = (cells_d * ws.p + kCoefPad) * sizeof(double2), bf = (cells_f * ws.p + kCoefPad) * sizeof(float2);
    for (double2 *m : {ws.mp_d, ws.mp2_d})
        if (m) launch_zero(m, bd, s);
    for (float2 *m : {ws.mp_f, ws.mp2_f})
        if (m && cells_f > 0) launch_zero(m, bf, s);
    HIP_TRY(hipGetLastError());
    return FMM_OK;
}

int ensure_workspace(fmm_tree *t, int p, int precision, bool backward, hipStream_t s)
{
    Workspace &ws = *t->wsp;
    const int split = split_level(t, precision);
    const int L = t->depth;
    if (ws.p != p || ws.precision != precision || ws.split != split) {
        hipError_t e = hipDeviceSynchronize();
        if (e != hipSuccess) return hip_fail(e, "hipDeviceSynchronize");
        free_workspace(ws);
    }
    const int64_t n = t->n;
    const int64_t cells_d = level_base(std::min(split, L) + 1);
    const int64_t cells_f = level_base(L + 1) - cells_d;
    const size_t gam_bytes = precision == FMM_FP64 ? sizeof(double) : sizeof(float);
    int rc = FMM_OK;
    if (!ws.gam) {
        if ((rc = dev_alloc_block((char **)&ws.gam, n * gam_bytes, "circulations in tree order"))) return rc;
        if ((rc = dev_alloc_block(&ws.stage, n, "velocities in tree order"))) return rc;
        if ((rc = dev_alloc_block(&ws.near, n, "near field"))) return rc;
        if (L >= 2) {
            if ((rc = dev_alloc_block(&ws.mp_d, cells_d * p + kCoefPad, "multipoles"))) return rc;
            if ((rc = dev_alloc_block(&ws.lo_d, cells_d * p + kCoefPad, "locals"))) return rc;
            if (cells_f > 0) {
                if ((rc = dev_alloc_block(&ws.mp_f, cells_f * p + kCoefPad, "multipoles"))) return rc;
                if ((rc = dev_alloc_block(&ws.lo_f, cells_f * p + kCoefPad, "locals"))) return rc;
            }
            // Empty cells are never written; the MFMA M2L reads them as zero rows.
            HIP_TRY(hipMemsetAsync(ws.mp_d, 0, (cells_d * p + kCoefPad) * sizeof(double2), s));
            HIP_TRY(hipMemsetAsync(ws.lo_d, 0, (cells_d * p + kCoefPad) * sizeof(double2), s));
            if (cells_f > 0) {
                HIP_TRY(hipMemsetAsync(ws.mp_f, 0, (cells_f * p + kCoefPad) * sizeof(float2), s));
                HIP_TRY(hipMemsetAsync(ws.lo_f, 0, (cells_f * p + kCoefPad) * sizeof(float2), s));
            }
        }
        ws.p = p;
        ws.precision = precision;
        ws.split = split;
        ws.owner = t->serial;  // zeroed just now
    }
    if (!ws.sums) {
        // the mutual slots, or the adjoint sums at 256-byte aligned offsets 0, A(32n)
        auto a256 = [](size_t b) { return (b + 255) / 256 * 256; };
        const size_t nn = (size_t)n;
        const size_t o_src = a256(32 * nn);
        const size_t bytes = std::max(9 * nn * (precision == FMM_FP64 ? 16 : 8), o_src + 32 * nn);
        if ((rc = dev_alloc_block((char **)&ws.sums, bytes, "near-field sums"))) return rc;
        ws.sums_bytes = bytes;
        ws.slots = ws.sums;
        ws.bwd_near = (double4 *)ws.sums;
        ws.bwd_src = (double4 *)((char *)ws.sums + o_src);
    }
    if (backward && !ws.adj) {
        auto adjoint_arrays = [&]() -> int {
            if ((rc = dev_alloc_block(&ws.adj, n, "adjoint charges"))) return rc;
            if (precision != FMM_FP64 && (rc = dev_alloc_block((float2 **)&ws.rec2, n, "adjoint charges (FP32)"))) return rc;
            if (L < 2) return FMM_OK;
            // the far field of the charges q, computed beside that of the charges c
            if ((rc = dev_alloc_block(&ws.mp2_d, cells_d * p + kCoefPad, "adjoint multipoles"))) return rc;
            if ((rc = dev_alloc_block(&ws.lo2_d, cells_d * p + kCoefPad, "adjoint locals"))) return rc;
            HIP_TRY(hipMemsetAsync(ws.mp2_d, 0, (cells_d * p + kCoefPad) * sizeof(double2), s));
            if (cells_f > 0) {
                if ((rc = dev_alloc_block(&ws.mp2_f, cells_f * p + kCoefPad, "adjoint multipoles"))) return rc;
                if ((rc = dev_alloc_block(&ws.lo2_f, cells_f * p + kCoefPad, "adjoint locals"))) return rc;
                HIP_TRY(hipMemsetAsync(ws.mp2_f, 0, (cells_f * p + kCoefPad) * sizeof(float2), s));
            }
            return FMM_OK;
        };
        // whole or not at all (ws.adj tells the next call that the group is there)
        if ((rc = adjoint_arrays())) {
            (void)hipStreamSynchronize(s);
            auto drop = [](auto *&q) {
                block_free(q);
                q = nullptr;
            };
            drop(ws.adj);
            drop(ws.rec2);
            drop(ws.mp2_d);
            drop(ws.lo2_d);
            drop(ws.mp2_f);
            drop(ws.lo2_f);
            return rc;
        }
        // with them what the pair force needs beside the forward's arrays; without it the
        // separate sums serve
        if (!outputs_windowed(n, kForceRow)) {
            for (auto [q, bytes] : {std::pair{(void **)&ws.range, (kRangeBlocks + 1) * sizeof(double2)},
                                    std::pair{&ws.phi_slots, 9 * n * gam_bytes}})
                if (block_alloc(q, bytes) != hipSuccess) *q = nullptr;
        }
    }
    if (ws.owner != t->serial) {
        int rc2 = clear_multipoles(t, s);
        if (rc2) return rc2;
        ws.owner = t->serial;
    }
    return FMM_OK;
}

// A handle whose arrays are there (see fmm_tree::released).
int check_tree(const fmm_tree *t)
{
    if (!t) return fail(FMM_ESTATE, "null tree handle");
    if (t->released)
        return fail(FMM_ESTATE, "the tree's arrays were released by a failed rebuild: rebuild or destroy it");
    return FMM_OK;
}

int check_eval_args(fmm_tree *t, const double *gamma, double sigma, int p, int precision)
{
    if (int rc = check_tree(t)) return rc;
    if (!gamma) return fail(FMM_EINVAL, "gamma is NULL");
    if (!(sigma > 0.0) || !std::isfinite(sigma)) return fail(FMM_EINVAL, "sigma must be finite and > 0");
    if (p < 1 || p > kMaxP) return fail(FMM_EINVAL, "p must be in [1, 32]");
    if (precision != FMM_FP64 && precision != FMM_MIXED) return fail(FMM_EINVAL, "unknown precision");
    return FMM_OK;
}


// FMM_OPT_VALIDATE: the circulations (and the cotangent of an adjoint call) are checked
// for NaN and infinities before any other work of the call; a bad value gives FMM_EINVAL
// naming the lowest particle index.  The check synchronises the main stream.
int validate_inputs(fmm_tree *t, const double *gamma, const double *dl_duv, hipStream_t s)
{
    if (!t->validate) return FMM_OK;
    int64_t bad = -1;
    if (!t->d_flag)
        if (int rc = dev_alloc(&t->d_flag, 1, "input check flag")) return rc;
    HIP_TRY(find_nonfinite(gamma, t->n, 1, t->d_flag, s, bad));
    if (bad >= 0) return fail(FMM_EINVAL, "non-finite circulation (particle " + std::to_string(bad) + ")");
    if (dl_duv) {
        HIP_TRY(find_nonfinite(dl_duv, t->n, 2, t->d_flag, s, bad));
        if (bad >= 0) return fail(FMM_EINVAL, "non-finite dL/du (particle " + std::to_string(bad) + ")");
    }
    return FMM_OK;
}

FarArgs far_args(const fmm_tree *t, const Workspace &ws, int p, int precision, bool adjoint)
{
    FarArgs a{};
    a.t = t;
    a.p = p;
    a.split = ws.split;
    a.mp_d = adjoint ? ws.mp2_d : ws.mp_d;
    a.lo_d = adjoint ? ws.lo2_d : ws.lo_d;
    a.mp_f = adjoint ? ws.mp2_f : ws.mp_f;
    a.lo_f = adjoint ? ws.lo2_f : ws.lo_f;
    a.pos = t->d_pos[precision == FMM_FP64];
    a.gam = ws.gam;
    a.rec_is_double = precision == FMM_FP64;
    a.adj = adjoint ? ws.adj : nullptr;
    return a;
}

// Stage costs of the mixed form (p = 12..16) on one MI355X, in ms, set to the stages of
// serialised calls on uniform (2^18 to 2^22 particles, 4 and 16 per leaf) and patch trees
// (10^6 to 2^24), within 25% of each (the complexity terms of section "Complexity Estimates"
// with the counts a launch pays for):
//   T_near = kNear0 + kNearPair pairs + kNearVisit 9 N_leaves,
//   T_far  = kFar0 + kFarParticle n + kFarCell cells + kFarLevel L.
constexpr double kNear0 = 0.020, kNearPair = 2.3e-10, kNearVisit = 4.5e-8;
constexpr double kFar0 = 0.030, kFarParticle = 1.6e-8, kFarCell = 0.7e-6, kFarLevel = 0.006;

// The part of T_near that grows with the tree.
double near_work_ms(const fmm_tree *t)
{
    return kNearPair * (double)t->p2p_pairs + kNearVisit * 9.0 * (double)t->nonempty_leaves;
}

// Predicted far-field / near-field time of the tree (the model above).
double far_near_ratio(const fmm_tree *t)
{
    double cells = 0;
    for (int l = 2; l <= t->depth; ++l) cells += (double)t->list_len[l];
    const double near = kNear0 + near_work_ms(t);
    const double far = kFar0 + kFarParticle * (double)t->n + kFarCell * cells + kFarLevel * t->depth;
    return far / near;
}

// Whether a call runs the far chain beside the near field (FMM_OPT_SCHEDULE 0), after it
// (1), or by the model (2, the default): both are throughput work on the same CUs.
//  - A near field of less than kSerialNear ms of work is not worth the second stream: the
//    events between the streams cost about 25 us (uniform 4096 particles, depth 4, FP64: 53 us
//    serialised against 85-94 overlapped; 50021, depth 6: 77 against 94-100; 2^18, depth 7,
//    mixed: 139 against 152-166).
//  - In the mixed form calls beyond a far/near ratio of kSerialRatio are serialised: there is
//    too little near field to run beside.  Up to 2.4 the best cap still gained (uniform 2^22,
//    depth 10: 2.44 against 2.56 ms).
//  - FP64 calls overlap (1024^2 lattice: 0.347 against 0.390 ms in a row of calls, 0.40 against 0.41
//    alone and in the first twenty after a pause; 2^21 uniform, depth 9: 0.91 against 1.03).
constexpr double kSerialRatio = 4.0, kSerialNear = 0.020;
bool call_overlaps(const fmm_tree *t, int precision)
{
    if (t->schedule != 2) return t->schedule == 0;
    if (t->depth < 2) return true;
    if (near_work_ms(t) < kSerialNear) return false;
    return precision == FMM_FP64 || far_near_ratio(t) <= kSerialRatio;
}

// Near-field occupancy cap of a call (FMM_OPT_NEAR_OCCUPANCY), automatic from the tree: the far
// chain takes the slots the cap leaves.  By the predicted far/near ratio r and near-field time T
// (best cap in brackets, from all caps on 40 trees):
//  - r < 0.05: none (2^24 patch particles at depth 9, mixed: 21.1 ms uncapped, 21.6 at six,
//    26.7 at three);
//  - mixed, r < 0.3 or T >= 0.25 ms: six (2^24 patches at depth 10: 7.47 ms [7.45], 2^23 at
//    depth 9: 5.94, 5.98 uncapped, 7.34 at three; uniform 2^22 at depth 10: 1.57 against 1.68 at
//    four and 2.02 at three, at depth 9: 0.777 against 0.831 and 0.958);
//  - mixed, T >= 0.1 ms: five for r < 1 (2^20 uniform at depth 7: 0.261 [0.255 at six]), else
//    four (2^21 uniform at depth 9: 0.482, 0.505 at five, 0.581 at three);
//  - mixed, smaller: three for r < 2.2 (2^20 uniform at depth 8: 0.230, 0.240 at five), else two
//    (2^19 at depth 8: 0.195, 0.204 at three and at six);
//  - FP64 (at most 5 wavefronts per SIMD), r < 1.2: four (2^21 patches at depth 9: 1.62 ms, 1.69
//    at three and uncapped; 4 10^5 at depth 7: 0.565, 0.600 and 0.571), else three (1024^2
//    lattice, depth 8, p = 12: 0.364, 0.380 at four, 0.413 at two, 0.397 uncapped), two below
//    T = 0.05 ms (200003 uniform at depth 6, p = 24: 0.168, 0.176 at three, 0.206 uncapped);
//  - a work list of less than 4096 entries leaves slots free by itself: no cap.
int choose_occupancy(const fmm_tree *t, int precision, bool overlap)
{
    if (!overlap || t->depth < 2) return 0;
    if (t->near_occupancy >= 0) return t->near_occupancy;
    const int64_t entries = use_mutual(t) ? t->nnear_work : t->nunits;
    if (entries < 4096) return 0;
    const double r = far_near_ratio(t), near = kNear0 + near_work_ms(t);
    if (r < 0.05) return 0;
    if (precision == FMM_FP64) return r < 1.2 ? 4 : near < 0.05 ? 2 : 3;
    if (r < 0.3 || near >= 0.25) return 6;
    if (near >= 0.1) return r < 1.0 ? 5 : 4;
    return r < 2.2 ? 3 : 2;
}

// The same for the adjoint's pair force, whose kernels hold fewer wavefronts (FP32 six per SIMD,
// five with Phi; FP64 four and three) and take longer, beside its two far chains: mixed at most five,
// four with Phi (adjoint of 2^22 patch particles at depth 9: 3.66 ms at five, 3.71 at six; with
// dl_dgamma 4.50 at four, 4.59 at five), and one more than the forward where that is less (2^20
// uniform at depth 8: 0.397 ms at four, 0.420 at three; 2^19: 0.295 at three, 0.340 at two), FP64 one
// less than the forward (700001 patches at depth 8: 1.02 ms at three, 1.05 at four; 1024^2 lattice:
// 0.619 at two, 0.658 at three).
int choose_force_occupancy(const fmm_tree *t, int precision, bool overlap, bool phi)
{
    const int cap = choose_occupancy(t, precision, overlap);
    if (t->near_occupancy >= 0 || cap == 0) return cap;
    if (precision == FMM_FP64) return cap > 2 ? cap - 1 : cap;
    return cap < 4 ? cap + 1 : std::min(cap, phi ? 4 : 5);
}

// Whether the pair force's FP32 sums are at least as near to 64-bit sums as the separate sums
// (see p2p_force_kernel): not where the option makes smaller leaves dense than by default (up to
// 1.55 times their error at 4 particles per leaf, 1.04 at 24, 0.98 at 32), nor where target-centric
// units meet leaves of several tiles, whose sums the separate ones fold leaf by leaf (1.03).  FP64:
// always.
constexpr int kForceDense = 32;
bool force_accurate(const fmm_tree *t, int precision)
{
    return precision == FMM_FP64 || (use_mutual(t) ? t->dense_leaf >= kForceDense : t->max_leaf <= 64);
}

struct Timing {
    std::array<hipEvent_t, kNumEvents> ev{};
    bool on = false;
    int init(fmm_tree *t)
    {
        on = t->timing != 0;
        if (!on) return FMM_OK;
        for (auto &e : ev) HIP_TRY(hipEventCreate(&e));
        return FMM_OK;
    }
    void mark(int k, hipStream_t s)
    {
        if (on) hipEventRecord(ev[k], s);
    }
};

// The tree's leaf-unit coordinates in the precision of a call, made on its first use.
int ensure_positions(fmm_tree *t, int precision, hipStream_t s)
{
    const int d = precision == FMM_FP64;
    if (t->d_pos[d]) return FMM_OK;
    if (!t->pos_buf[d]) {
        const int rc = dev_alloc_async((char **)&t->pos_buf[d], (size_t)t->n * (d ? sizeof(double2) : sizeof(float2)),
                                       "leaf-unit coordinates", s);
        if (rc) return rc;
    }
    t->d_pos[d] = t->pos_buf[d];
    launch_leaf_coords(t, d, t->d_pos[d], s);
    return FMM_OK;
}

// The per-call arrays of an evaluation carved from the static workspace (no allocation):
// circulations, staged velocities, near field, leaf-unit coordinates (in `sums`, when the
// tree has none yet), slots (mutual form), then the multipoles and locals of every level,
// each 256-byte aligned.  A mixed call for which they do not fit with levels 2..5 in FP64 (20 KiB
// per term) takes L_c as it stands.  FMM_EINVAL when that does not fit, naming both sizes.
int static_ws(const fmm_tree *t, int p, int precision, Workspace &ws)
{
    char *base = nullptr;
    const int e = static_workspace(t->device, &base);
    if (e != 0) return hip_fail((hipError_t)e, "looking up the static workspace");
    const int L = t->depth;
    const int64_t n = t->n;
    const size_t real = precision == FMM_FP64 ? sizeof(double) : sizeof(float);
    const size_t slot = precision == FMM_FP64 ? sizeof(double2) : sizeof(float2);
    auto carve = [&](int split) {
        const int64_t cells_d = L >= 2 ? level_base(std::min(split, L) + 1) * p + kCoefPad : 0;
        const int64_t cells_f = L >= 2 && level_base(L + 1) > level_base(std::min(split, L) + 1)
                                    ? (level_base(L + 1) - level_base(std::min(split, L) + 1)) * p + kCoefPad
                                    : 0;
        size_t off = 0;
        auto take = [&](size_t bytes) {
            const size_t at = off;
            off += (bytes + 255) / 256 * 256;
            return base + at;
        };
        ws = Workspace{};
        ws.p = p;
        ws.precision = precision;
        ws.split = split;
        ws.gam = take((size_t)n * real);
        ws.stage = (double2 *)take((size_t)n * sizeof(double2));
        ws.near = (double2 *)take((size_t)n * sizeof(double2));
        // the tree's leaf-unit coordinates when an allocating evaluation has not made them yet
        if (!t->d_pos[precision == FMM_FP64]) ws.sums = take((size_t)n * 2 * real);
        if (use_mutual(t)) ws.slots = take((size_t)9 * n * slot);
        ws.mp_d = (double2 *)take((size_t)cells_d * sizeof(double2));
        ws.lo_d = (double2 *)take((size_t)cells_d * sizeof(double2));
        ws.mp_f = (float2 *)take((size_t)cells_f * sizeof(float2));
        ws.lo_f = (float2 *)take((size_t)cells_f * sizeof(float2));
        return off;
    };
    size_t bytes = carve(split_level(t, precision));
    if (bytes > kStaticWorkspaceBytes && precision != FMM_FP64) bytes = carve(std::min(t->lc, L));
    if (bytes > kStaticWorkspaceBytes)
        return fail(FMM_EINVAL, "this evaluation needs " + std::to_string(bytes) + " bytes of device workspace, more "
                                "than the " + std::to_string(kStaticWorkspaceBytes) + " bytes of the static workspace");
    return FMM_OK;
}

// Stages 4-10.  noalloc: the per-call arrays in the static workspace (cleared where they
// must start at zero) and the tables already on the device; no allocation, no events.
int run_forward(fmm_tree *t, const double *gamma, double sigma, int p, int precision, void *main_stream,
                void *side_stream, double *uv, double *uv_near, double *uv_far, const double *base = nullptr,
                double h = 0.0, bool noalloc = false)
{
    int rc = check_eval_args(t, gamma, sigma, p, precision);
    if (rc) return rc;
    if (!uv && !(uv_near && uv_far)) return fail(FMM_EINVAL, "output is NULL");
    BusyGuard guard(t);
    if (!guard.ok) return fail(FMM_ESTATE, "tree handle in use by another thread");
    HIP_TRY(hipSetDevice(t->device));
    hipStream_t ms = (hipStream_t)main_stream;
    if ((rc = validate_inputs(t, gamma, nullptr, ms))) return rc;
    std::string err;
    Workspace local;
    if (noalloc) {
        if ((rc = shared_tables(t->device, p, &t->tabs, err, false)))
            return fail(FMM_ESTATE, err + " (an allocating evaluation with this p makes them)");
        if ((rc = static_ws(t, p, precision, local))) return rc;
        // multipoles of empty cells are read as zero rows by M2L
        if (local.mp_d) launch_zero(local.mp_d, (size_t)((char *)local.lo_d - (char *)local.mp_d), ms);
        if (local.mp_f) launch_zero(local.mp_f, (size_t)((char *)local.lo_f - (char *)local.mp_f), ms);
        if (local.sums) launch_leaf_coords(t, precision == FMM_FP64, local.sums, ms);
    } else {
        if ((rc = shared_tables(t->device, p, &t->tabs, err)))
            return fail(rc == -2 ? FMM_ENOMEM : FMM_EDEVICE, err);
        if ((rc = ensure_workspace(t, p, precision, false, ms)) || (rc = ensure_positions(t, precision, ms)))
            return rc;
    }
    Workspace &ws = noalloc ? local : *t->wsp;
    const void *pos = noalloc && local.sums ? local.sums : t->d_pos[precision == FMM_FP64];

    hipStream_t ss = side_stream ? (hipStream_t)side_stream : t->aux.stream;
    const bool overlap = call_overlaps(t, precision);
    if (!overlap) ss = ms;
    const double alpha = record_alpha(sigma, precision);
    const int is_double = precision == FMM_FP64;
    FarArgs a = far_args(t, ws, p, precision, false);
    a.pos = pos;
    a.gam = nullptr;  // P2M starts before the circulations are gathered: it reads the staging array
    t->occupancy_in_use = choose_occupancy(t, precision, overlap);
    a.no_lds = t->occupancy_in_use > 0;
    Timing tm;
    if (!noalloc && (rc = tm.init(t))) return rc;

    tm.mark(0, ms);
    a.gamma = launch_stage_in(t, gamma, kForwardRow, ms);
    if (overlap) {  // the far chain needs only the staged circulations: it starts beside pack
        HIP_TRY(hipEventRecord(t->aux.fork, ms));
        HIP_TRY(hipStreamWaitEvent(ss, t->aux.fork, 0));
    }
    launch_pack(t, a.gamma, is_double, ws.gam, ms);
    tm.mark(1, ms);
    tm.mark(2, ss);
    launch_far_chain(a, ss);
    tm.mark(3, ss);
    if (overlap) HIP_TRY(hipEventRecord(t->aux.join, ss));
    void *slots = use_mutual(t) ? ws.slots : nullptr;
    tm.mark(4, ms);
    launch_p2p_forward(t, pos, ws.gam, is_double, alpha, ws.near, slots, ms);
    tm.mark(5, ms);
    if (overlap) HIP_TRY(hipStreamWaitEvent(ms, t->aux.join, 0));
    tm.mark(6, ms);
    launch_finalize(t, a, ws.near, slots, is_double, alpha, uv, uv_near, uv_far, ws.stage, base, h, ms);
    tm.mark(7, ms);
    HIP_TRY(hipGetLastError());
    if (tm.on) t->pending_timing.push_back(tm.ev);
    return FMM_OK;
}

}  // namespace

namespace {

// Argument checks shared by both builds; a new tree with device facts filled in.
int new_tree(const double *xy, int64_t n, int depth, const double *root_box, fmm_tree **out, fmm_tree *&t)
{
    g_last_error.clear();
    t = nullptr;
    if (!out) return fail(FMM_EINVAL, "out is NULL");
    *out = nullptr;
    if (!xy) return fail(FMM_EINVAL, "xy is NULL");
    if (n < 1 || n >= (int64_t(1) << 31)) return fail(FMM_EINVAL, "n must be in [1, 2^31)");
    if (depth < 1 || depth > kMaxDepth) return fail(FMM_EINVAL, "depth must be in [1, 12]");
    if (root_box && (!std::isfinite(root_box[0]) || !std::isfinite(root_box[1]) || !(root_box[2] > 0.0) ||
                     !std::isfinite(root_box[2])))
        return fail(FMM_EINVAL, "root_box must be finite with side > 0");
    int dev = 0;
    const hipError_t de = hipGetDevice(&dev);
    if (de != hipSuccess) return hip_fail(de, "hipGetDevice");
    retain_pool(dev);
    t = new fmm_tree();
    static std::atomic<uint64_t> next_serial{1};
    t->serial = next_serial.fetch_add(1);
    t->device = dev;
    int cus = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1) cus = 256;
    t->num_cus = cus;
    t->n = n;
    t->depth = depth;
    return FMM_OK;
}

// Common end of both builds: the tree's side stream and events.
int finish_tree(fmm_tree *t)
{
    if (!t->aux.stream) {
        const hipError_t e = side_stream_take(t->device, t->aux);
        if (e != hipSuccess) return hip_fail(e, "creating stream/events");
    }
    return FMM_OK;
}

}  // namespace

// ---------------------------------------------------------------------------------------
// Stages 1-3: tree construction, binning, work lists -- on the device (default) or on
// the host (reference build; both give identical trees)
// ---------------------------------------------------------------------------------------
namespace {

// The device build; the options of `opts` (a tree being replaced) are taken over before
// the near-field plan is made, since that plan depends on them.  arena: device memory
// idle during the build that its temporaries may use; after_checks(new tree): see
// build_tree_device.
int build_device(const double *xy, int64_t n, int depth, const double *root_box, void *stream, const fmm_tree *opts,
                 fmm_tree **out, BuildArena *arena = nullptr,
                 const std::function<void(fmm_tree *)> &after_checks = {})
{
    fmm_tree *t = nullptr;
    int rc = new_tree(xy, n, depth, root_box, out, t);
    if (rc) return rc;
    if (opts) {
        t->lc = opts->lc;
        t->schedule = opts->schedule;
        t->near_mutual = opts->near_mutual;
        t->dense_leaf = opts->dense_leaf;
        t->near_occupancy = opts->near_occupancy;
        t->timing = opts->timing;
        t->validate = opts->validate;
    }
    hipStream_t s = (hipStream_t)stream;
    std::string err;
    int64_t bad = -1;
    {
        BuildArenaScope scope(arena);
        rc = build_tree_device(t, xy, root_box, s, err, bad, [&]() {
            if (after_checks) after_checks(t);
        });
        if (!rc) rc = finish_tree(t);
        else {
            if (bad >= 0) err += " (particle " + std::to_string(bad) + ")";
            fail(rc, err);
        }
    }
    if (!rc) {
        const hipError_t e = hipDeviceSynchronize();
        if (e != hipSuccess) rc = hip_fail(e, "hipDeviceSynchronize");
    }
    if (rc) {
        free_tree(t);
        return rc;
    }
    bound_idle(t->device);  // (arrays that had to grow)
    *out = t;
    return FMM_OK;
}

}  // namespace

extern "C" int fmm_build_tree(const double *xy, int64_t n, int depth, const double *root_box, void *stream,
                              fmm_tree **out)
{
    return build_device(xy, n, depth, root_box, stream, nullptr, out);
}

extern "C" int fmm_rebuild_tree(fmm_tree *prev, const double *xy, int64_t n, const double *root_box, void *stream,
                                fmm_tree **out)
{
    g_last_error.clear();
    if (out) *out = nullptr;
    if (!prev) return fail(FMM_ESTATE, "null tree handle");
    if (n != prev->n) return fail(FMM_EINVAL, "n must equal the particle count of the tree being rebuilt");
    int dev = 0;
    HIP_TRY(hipGetDevice(&dev));
    if (dev != prev->device) return fail(FMM_EINVAL, "the current device is not the tree's");
    BusyGuard guard(prev);
    if (!guard.ok) return fail(FMM_ESTATE, "tree is in use by another call");
    // Earlier calls on prev, or on a tree sharing its workspace, may still use the
    // workspace and prev's arrays.
    HIP_TRY(hipDeviceSynchronize());
    // One tree's arrays at a time: the build's temporaries go to the workspace's per-call
    // region (idle between calls), and prev's arrays pass to the new tree once the positions
    // have passed their checks (those of a host build are released there).
    BuildArena arena;
    arena.base = (char *)prev->wsp->sums;
    arena.cap = prev->wsp->sums ? prev->wsp->sums_bytes : 0;
    hipStream_t s = (hipStream_t)stream;
    auto hand_over = [prev, s](fmm_tree *t) {
        if (prev->pooled) take_over_arrays(t, prev);
        else release_tree_arrays(prev, s);
        prev->released = true;
    };
    fmm_tree *t = nullptr;
    int rc = build_device(xy, n, prev->depth, root_box, stream, prev, &t, &arena, hand_over);
    if (rc) return rc;
    std::swap(t->wsp, prev->wsp);
    t->wsp->owner = kForeignOwner;  // cleared by the next call
    std::swap(t->d_flag, prev->d_flag);
    guard.release();
    free_tree(prev);
    *out = t;
    return FMM_OK;
}

extern "C" int fmm_build_tree_host(const double *xy, int64_t n, int depth, const double *root_box, void *stream,
                                   fmm_tree **out)
{
    fmm_tree *t = nullptr;
    int rc0 = new_tree(xy, n, depth, root_box, out, t);
    if (rc0) return rc0;
    try {
        hipStream_t s = (hipStream_t)stream;
        std::vector<double> h(2 * (size_t)n);
        hipError_t e = hipMemcpyAsync(h.data(), xy, h.size() * sizeof(double), hipMemcpyDeviceToHost, s);
        if (e == hipSuccess) e = hipStreamSynchronize(s);
        if (e != hipSuccess) {
            free_tree(t);
            return hip_fail(e, "copying positions to the host");
        }
        UniformHostTree ht;
        int64_t bad = -1;
        std::string err;
        int rc = build_host_tree(h.data(), n, depth, root_box, ht, bad, err);
        if (rc) {
            free_tree(t);
            return fail(rc, err);
        }
        t->x0 = ht.x0;
        t->y0 = ht.y0;
        t->side = ht.side;
        t->stage_shift = ht.stage_shift;
        t->list_off = ht.list_off;
        t->list_len = ht.list_len;
        t->class_off = ht.class_off;
        t->p2p_pairs = ht.p2p_pairs;
        t->m2l_pairs = ht.m2l_pairs;
        t->nonempty_leaves = ht.nonempty_leaves;
        t->max_leaf = ht.max_leaf;
        t->nunits = (int64_t)ht.units.size();
        if (!rc) rc = upload(&t->d_perm, ht.perm, "permutation");
        if (!rc) rc = upload(&t->d_gpos1, ht.gpos1, "staging slots");
        if (!rc) rc = upload(&t->d_gpos2, ht.gpos2, "staging slots");
        if (!rc) rc = dev_alloc(&t->d_st1, n, "staging array");
        if (!rc) rc = upload(&t->d_leaf_of, ht.leaf_of, "leaf ids");
        if (!rc) rc = upload_as(&t->d_xy, ht.xy, "sorted positions");
        if (!rc) rc = upload(&t->d_leaf_start, ht.leaf_start, "leaf offsets");
        if (!rc) rc = upload(&t->d_counts, ht.counts, "cell counts");
        if (!rc) rc = upload(&t->d_lists, ht.lists, "cell lists");
        if (!rc) rc = upload_as(&t->d_units, ht.units, "P2P work units");
        if (!rc) rc = upload(&t->d_tile_start, ht.tile_start, "tile offsets");
        if (!rc) rc = upload_as(&t->d_tile_box, ht.tile_box, "tile boxes");
        if (!rc) rc = finish_tree(t);
        std::string plan_err;
        if (!rc && (rc = build_near_plan_device(t, s, plan_err))) fail(rc, plan_err);
        if (rc) {
            free_tree(t);
            return rc;
        }
    } catch (const std::bad_alloc &) {
        if (t) free_tree(t);
        return fail(FMM_ENOMEM, "host allocation failed while building the tree");
    }
    *out = t;
    return FMM_OK;
}

extern "C" int fmm_share_workspace(fmm_tree *t, fmm_tree *from)
{
    g_last_error.clear();
    if (!t || !from) return fail(FMM_ESTATE, "null tree handle");
    if (t == from) return FMM_OK;
    if (t->n != from->n || t->depth != from->depth || t->device != from->device)
        return fail(FMM_EINVAL, "trees sharing a workspace need the same n, depth and device");
    BusyGuard g1(t);
    if (!g1.ok) return fail(FMM_ESTATE, "tree is in use by another call");
    BusyGuard g2(from);
    if (!g2.ok) return fail(FMM_ESTATE, "tree is in use by another call");
    if (t->wsp == from->wsp) return FMM_OK;
    HIP_TRY(hipSetDevice(t->device));
    HIP_TRY(hipDeviceSynchronize());  // t's earlier calls may still use its workspace
    if (t->wsp.use_count() == 1) free_workspace(*t->wsp);
    t->wsp = from->wsp;
    return FMM_OK;
}

extern "C" int fmm_tree_info(const fmm_tree *t, int64_t *n, int *depth, double *root_box, int64_t *p2p_pairs,
                             int64_t *m2l_pairs, int64_t *nonempty_leaves, int64_t *max_leaf)
{
    if (int rc = check_tree(t)) return rc;
    if (n) *n = t->n;
    if (depth) *depth = t->depth;
    if (root_box) {
        root_box[0] = t->x0;
        root_box[1] = t->y0;
        root_box[2] = t->side;
    }
    if (p2p_pairs) *p2p_pairs = t->p2p_pairs;
    if (m2l_pairs) *m2l_pairs = t->m2l_pairs;
    if (nonempty_leaves) *nonempty_leaves = t->nonempty_leaves;
    if (max_leaf) *max_leaf = t->max_leaf;
    return FMM_OK;
}

namespace fmm {
void launch_widen_perm(const fmm_tree *t, int64_t *perm, int32_t *leaf, hipStream_t s);
}

extern "C" int fmm_tree_levels(const fmm_tree *t, int64_t *nonempty, int max_levels)
{
    if (int rc = check_tree(t)) return rc;
    if (!nonempty || max_levels < 1) return fail(FMM_EINVAL, "nonempty is NULL or max_levels < 1");
    std::vector<int> h((size_t)level_base(std::min(t->depth, 1) + 1));
    for (int l = 0; l < max_levels; ++l) nonempty[l] = 0;
    // levels 0 and 1 from the cell counts (they hold no expansions and have no list)
    const int top = std::min(t->depth, 1);
    if (hipMemcpy(h.data(), t->d_counts, h.size() * sizeof(int), hipMemcpyDeviceToHost) != hipSuccess)
        return fail(FMM_EDEVICE, "reading cell counts");
    for (int l = 0; l <= top && l < max_levels; ++l)
        for (int64_t c = level_base(l); c < level_base(l + 1); ++c) nonempty[l] += h[c] > 0;
    for (int l = 2; l <= t->depth && l < max_levels; ++l) nonempty[l] = t->list_len[l];
    return FMM_OK;
}

extern "C" int fmm_tree_permutation(const fmm_tree *t, int64_t *perm, int32_t *leaf, void *stream)
{
    if (int rc = check_tree(t)) return rc;
    if (!perm) return fail(FMM_EINVAL, "perm is NULL");
    HIP_TRY(hipSetDevice(t->device));
    launch_widen_perm(t, perm, leaf, (hipStream_t)stream);
    HIP_TRY(hipGetLastError());
    return FMM_OK;
}

extern "C" int fmm_velocity(fmm_tree *t, const double *gamma, double sigma, int p, int precision,
                            void *main_stream, void *side_stream, double *uv)
{
    g_last_error.clear();
    if (!uv) return fail(FMM_EINVAL, "uv is NULL");
    return run_forward(t, gamma, sigma, p, precision, main_stream, side_stream, uv, nullptr, nullptr);
}

extern "C" int fmm_velocity_noalloc(fmm_tree *t, const double *gamma, double sigma, int p, int precision,
                                    void *main_stream, void *side_stream, double *uv)
{
    g_last_error.clear();
    if (!uv) return fail(FMM_EINVAL, "uv is NULL");
    return run_forward(t, gamma, sigma, p, precision, main_stream, side_stream, uv, nullptr, nullptr, nullptr, 0.0,
                       true);
}

extern "C" int fmm_velocity_parts(fmm_tree *t, const double *gamma, double sigma, int p, int precision,
                                  void *main_stream, void *side_stream, double *uv_near, double *uv_far)
{
    g_last_error.clear();
    if (!uv_near || !uv_far) return fail(FMM_EINVAL, "uv_near / uv_far is NULL");
    return run_forward(t, gamma, sigma, p, precision, main_stream, side_stream, nullptr, uv_near, uv_far);
}

namespace {

// The arrays of the pair force: the forward's near-field array and slots, with Phi the staging
// array and slots of its own, in FP32 the block maxima.  False (the separate sums then serve)
// if device memory did not hold them.
bool force_arrays(const fmm_tree *t, const Workspace &ws, bool phi, ForceNear &near)
{
    const bool mutual = use_mutual(t);
    if (!ws.range || (phi && mutual && !ws.phi_slots)) return false;
    near.near = ws.near;
    near.mask = mutual ? t->d_leaf_mask : nullptr;
    near.slots = mutual ? ws.slots : nullptr;
    near.phi = phi ? (double *)ws.stage : nullptr;  // free between pack and finalize
    near.phi_slots = phi && mutual ? ws.phi_slots : nullptr;
    return true;
}

// The adjoint of stages 4-10 for the cotangent scale * cot (user order), written as `out`
// says (see AdjointOut).
int run_backward(fmm_tree *t, const double *gamma, double sigma, int p, int precision, const double *cot,
                 double scale, void *main_stream, void *side_stream, const AdjointOut &out)
{
    int rc = check_eval_args(t, gamma, sigma, p, precision);
    if (rc) return rc;
    if (!cot) return fail(FMM_EINVAL, "dl_duv is NULL");
    if (!std::isfinite(scale)) return fail(FMM_EINVAL, "the cotangent scale must be finite");
    if (!out.dg && !out.dxe && !out.dxs && !out.dxy) return FMM_OK;
    BusyGuard guard(t);
    if (!guard.ok) return fail(FMM_ESTATE, "tree handle in use by another thread");
    HIP_TRY(hipSetDevice(t->device));
    if ((rc = validate_inputs(t, gamma, cot, (hipStream_t)main_stream))) return rc;
    std::string err;
    if ((rc = shared_tables(t->device, p, &t->tabs, err))) return fail(rc == -2 ? FMM_ENOMEM : FMM_EDEVICE, err);
    if ((rc = ensure_workspace(t, p, precision, true, (hipStream_t)main_stream)) ||
        (rc = ensure_positions(t, precision, (hipStream_t)main_stream)))
        return rc;
    Workspace &ws = *t->wsp;
    const bool need_src = out.dxs || out.dxy;
    const void *pos = t->d_pos[precision == FMM_FP64];

    hipStream_t ms = (hipStream_t)main_stream;
    hipStream_t ss = side_stream ? (hipStream_t)side_stream : t->aux.stream;
    const double alpha = record_alpha(sigma, precision);
    const int is_double = precision == FMM_FP64;
    // The pair force gives dl_dxy without its two parts, in half the near field's time over dense
    // leaves.  Where the outputs outgrow the last-level cache the separate sums stay, for their bits
    // and not for their time: there a step's adjoint has the bits of velocity_backward's parts added
    // up, which callers compare.  It costs 2^23 patch particles 18.4 against 11.7 ms at depth 9 and
    // 7.4 against 5.3 at depth 10, 2^24 at depth 10 23.4 against 15.9 (with dl_dgamma 23.7 against
    // 19.4), 2^24 uniform 7.10 against 6.76.
    ForceNear near;
    const bool force = out.dxy && !out.dxe && !out.dxs && !outputs_windowed(t->n, kForceRow) &&
                       force_accurate(t, precision) && force_arrays(t, ws, out.dg != nullptr, near);
    // The two far chains (the charges c: the derivative of their local expansion; the charges q:
    // the transpose pass A^T q = -A q) go through the same launches.  The pair force runs beside
    // them; the separate sums, which hold every wavefront slot, follow them.
    const bool overlap = force && call_overlaps(t, precision);
    if (!overlap) ss = ms;
    t->occupancy_in_use = choose_force_occupancy(t, precision, overlap, out.dg != nullptr);
    FarArgs fc = far_args(t, ws, p, precision, false);
    fc.no_lds = t->occupancy_in_use > 0;
    const FarArgs fq = far_args(t, ws, p, precision, true);
    Timing tm;
    if ((rc = tm.init(t))) return rc;

    tm.mark(0, ms);
    fc.gamma = launch_stage_in(t, gamma, kAdjointRow, ms);
    launch_pack(t, fc.gamma, is_double, ws.gam, ms);
    double *qscale = nullptr;
    if (force && !is_double) {
        launch_adjoint_range(t->n, gamma, cot, scale, ws.range, ms);
        near.qscale = qscale = (double *)(ws.range + kRangeBlocks);
    }
    launch_pack_adjoint(t, cot, scale, ws.adj, ws.rec2, is_double, ws.stage, qscale ? ws.range : nullptr, qscale,
                        ms);  // stage: free until finalize
    tm.mark(1, ms);
    if (overlap) {
        HIP_TRY(hipEventRecord(t->aux.fork, ms));
        HIP_TRY(hipStreamWaitEvent(ss, t->aux.fork, 0));
    }
    tm.mark(2, ss);
    launch_far_chain(fc, ss, &fq);
    tm.mark(3, ss);
    if (overlap) HIP_TRY(hipEventRecord(t->aux.join, ss));
    tm.mark(4, ms);
    const void *qv = is_double ? (const void *)ws.adj : ws.rec2;
    if (force) {
        launch_p2p_force(t, pos, ws.gam, qv, ws.adj, fc.gamma, is_double, alpha, near, ms);
        tm.mark(5, ms);
        if (overlap) HIP_TRY(hipStreamWaitEvent(ms, t->aux.join, 0));
        tm.mark(6, ms);
        launch_finalize_force(t, fc, fq, ws.adj, near, is_double, alpha, out, ms);
        tm.mark(7, ms);
        HIP_TRY(hipGetLastError());
        if (tm.on) t->pending_timing.push_back(tm.ev);
        return FMM_OK;
    }
    launch_p2p_backward(t, pos, ws.gam, qv, is_double, alpha, ws.bwd_near,
                        need_src ? ws.bwd_src : nullptr, ms);
    tm.mark(5, ms);
    tm.mark(6, ms);
    // once the outputs fill the last-level cache they reach user order through staging slots, kept in
    // arrays this call no longer reads: dL/dGamma in the FP32 charges (mixed) or the FP64
    // circulations, the evaluation part in the forward's staged velocities, the source part
    // in the forward's near-field array
    const int64_t out_bytes = (out.dg ? 8 : 0) + ((out.dxe || out.dxy) ? 16 : 0) + ((out.dxs || out.dxy) ? 16 : 0);
    const bool staged = outputs_windowed(t->n, out_bytes);
    double *st_g = !staged ? nullptr : is_double ? (double *)ws.gam : (double *)ws.rec2;
    double *st_x = staged ? (double *)ws.stage : nullptr;
    double *st_s = staged ? (double *)ws.near : nullptr;
    launch_finalize_backward(t, fc, fq, ws.bwd_near, ws.adj, ws.bwd_src, is_double, alpha, out, st_g, st_x,
                             st_s, ms);
    tm.mark(7, ms);
    HIP_TRY(hipGetLastError());
    if (tm.on) t->pending_timing.push_back(tm.ev);
    return FMM_OK;
}

}  // namespace

extern "C" int fmm_velocity_backward(fmm_tree *t, const double *gamma, double sigma, int p, int precision,
                                     const double *dl_duv, void *main_stream, void *side_stream, double *dl_dgamma,
                                     double *dl_dxeval, double *dl_dxsrc, double *dl_dxy)
{
    g_last_error.clear();
    AdjointOut out;
    out.dg = dl_dgamma;
    out.dxe = dl_dxeval;
    out.dxs = dl_dxsrc;
    out.dxy = dl_dxy;
    return run_backward(t, gamma, sigma, p, precision, dl_duv, 1.0, main_stream, side_stream, out);
}

extern "C" int fmm_transport_step(fmm_tree *t, const double *gamma, double sigma, int p, int precision,
                                  void *main_stream, void *side_stream, const double *x_base, double h, double *x_out)
{
    g_last_error.clear();
    if (!x_base || !x_out) return fail(FMM_EINVAL, "x_base / x_out is NULL");
    if (!std::isfinite(h)) return fail(FMM_EINVAL, "h must be finite");
    return run_forward(t, gamma, sigma, p, precision, main_stream, side_stream, x_out, nullptr, nullptr, x_base, h);
}

extern "C" int fmm_transport_vjp(fmm_tree *t, const double *gamma, double sigma, int p, int precision,
                                 const double *lam, double h, int flags, void *main_stream, void *side_stream,
                                 double *dl_dgamma, double *dl_dx)
{
    g_last_error.clear();
    if (flags & ~(FMM_ACC_GAMMA | FMM_ACC_X | FMM_IDENTITY)) return fail(FMM_EINVAL, "unknown flag");
    if (!lam) return fail(FMM_EINVAL, "lam is NULL");
    AdjointOut out;
    out.dg = dl_dgamma;
    out.dxy = dl_dx;
    out.lam = (flags & FMM_IDENTITY) ? lam : nullptr;
    out.acc_g = (flags & FMM_ACC_GAMMA) != 0;
    out.acc_xy = (flags & FMM_ACC_X) != 0;
    return run_backward(t, gamma, sigma, p, precision, lam, h, main_stream, side_stream, out);
}

extern "C" int fmm_set_option(fmm_tree *t, int key, int64_t value)
{
    if (!t) return fail(FMM_ESTATE, "null tree handle");
    switch (key) {
    case FMM_OPT_SCHEDULE:
        if (value < 0 || value > 2) return fail(FMM_EINVAL, "schedule must be 0, 1 or 2");
        t->schedule = (int)value;
        return FMM_OK;
    case FMM_OPT_COARSE_LEVEL:
        if (value < 1 || value > t->depth) return fail(FMM_EINVAL, "coarse level must be in [1, depth]");
        t->lc = (int)value;
        return FMM_OK;
    case FMM_OPT_NEAR_MUTUAL:
    case FMM_OPT_DENSE_LEAF: {
        if (key == FMM_OPT_NEAR_MUTUAL && value != 0 && value != 1)
            return fail(FMM_EINVAL, "near mutual must be 0 or 1");
        if (key == FMM_OPT_DENSE_LEAF && (value < 1 || value > (int64_t(1) << 30)))
            return fail(FMM_EINVAL, "dense leaf must be in [1, 2^30]");
        if (int rc = check_tree(t)) return rc;  // the plan is made from the tree's arrays
        HIP_TRY(hipSetDevice(t->device));
        HIP_TRY(hipDeviceSynchronize());  // the plan's arrays may be in use
        if (key == FMM_OPT_NEAR_MUTUAL) t->near_mutual = (int)value;
        else t->dense_leaf = (int)value;
        std::string err;
        const int rc = build_near_plan_device(t, t->aux.stream, err);
        return rc ? fail(rc, err) : FMM_OK;
    }
    case FMM_OPT_NEAR_OCCUPANCY:
        if (value < -1 || value > 8) return fail(FMM_EINVAL, "near occupancy must be in [-1, 8]");
        t->near_occupancy = (int)value;
        return FMM_OK;
    case FMM_OPT_TIMING:
        if (value != 0 && value != 1) return fail(FMM_EINVAL, "timing must be 0 or 1");
        t->timing = (int)value;
        return FMM_OK;
    case FMM_OPT_VALIDATE:
        if (value != 0 && value != 1) return fail(FMM_EINVAL, "validate must be 0 or 1");
        t->validate = (int)value;
        return FMM_OK;
    case 4:
    case 5:
        return fail(FMM_EINVAL, "option withdrawn (persistent near-field grid, far-field grid cap)");
    default:
        return fail(FMM_EINVAL, "unknown option");
    }
}

extern "C" int fmm_near_plan_info(const fmm_tree *t, int64_t *mutual_items, int64_t *mutual_pairs,
                                  int64_t *target_units)
{
    if (int rc = check_tree(t)) return rc;
    const bool m = use_mutual(t);
    if (mutual_items) *mutual_items = m ? t->nmut : 0;
    if (mutual_pairs) *mutual_pairs = m ? t->mutual_pairs : 0;
    if (target_units) *target_units = m ? t->nunits_tc : t->nunits;
    return FMM_OK;
}

extern "C" int fmm_get_timings(fmm_tree *t, double *ms, int64_t *calls)
{
    if (!t) return fail(FMM_ESTATE, "null tree handle");
    if (!ms) return fail(FMM_EINVAL, "ms is NULL");
    HIP_TRY(hipSetDevice(t->device));
    double acc[FMM_T_COUNT] = {};
    int64_t ncalls = 0;
    for (auto &ev : t->pending_timing) {
        HIP_TRY(hipEventSynchronize(ev[7]));
        HIP_TRY(hipEventSynchronize(ev[3]));
        float f;
        HIP_TRY(hipEventElapsedTime(&f, ev[0], ev[1]));
        acc[FMM_T_PACK] += f;
        HIP_TRY(hipEventElapsedTime(&f, ev[2], ev[3]));
        acc[FMM_T_FAR] += f;
        HIP_TRY(hipEventElapsedTime(&f, ev[4], ev[5]));
        acc[FMM_T_P2P] += f;
        HIP_TRY(hipEventElapsedTime(&f, ev[6], ev[7]));
        acc[FMM_T_FINAL] += f;
        HIP_TRY(hipEventElapsedTime(&f, ev[0], ev[7]));
        acc[FMM_T_TOTAL] += f;
        ++ncalls;
        for (auto e : ev) hipEventDestroy(e);
    }
    t->pending_timing.clear();
    for (int k = 0; k < FMM_T_COUNT; ++k) ms[k] = acc[k];
    if (calls) *calls = ncalls;
    return FMM_OK;
}

extern "C" int fmm_get_timeline(fmm_tree *t, double *ms, int count)
{
    if (!t) return fail(FMM_ESTATE, "null tree handle");
    if (!ms || count < 1) return fail(FMM_EINVAL, "ms is NULL or count < 1");
    if (t->pending_timing.empty()) return fail(FMM_ESTATE, "no call recorded with FMM_OPT_TIMING since the last read");
    HIP_TRY(hipSetDevice(t->device));
    auto &ev = t->pending_timing.back();
    HIP_TRY(hipEventSynchronize(ev[7]));
    HIP_TRY(hipEventSynchronize(ev[3]));
    for (int k = 0; k < count; ++k) {
        ms[k] = 0.0;
        if (k >= kNumEvents) continue;
        float f = 0.0f;
        HIP_TRY(hipEventElapsedTime(&f, ev[0], ev[k]));
        ms[k] = f;
    }
    return FMM_OK;
}

extern "C" void fmm_destroy_tree(fmm_tree *t)
{
    if (!t) return;
    hipSetDevice(t->device);
    hipDeviceSynchronize();
    free_tree(t);
}

int fmm::fail(int code, const std::string &msg)
{
    g_last_error = msg;
    return code;
}

void fmm::clear_last_error() { g_last_error.clear(); }

double fmm::record_alpha(double sigma, int precision)
{
    const double a = 1.0 / (sigma * std::sqrt(2.0));
    return precision == FMM_FP64 ? a : a * std::sqrt(1.4426950408889634073599246810019);
}

extern "C" const char *fmm_last_error(void) { return g_last_error.c_str(); }
