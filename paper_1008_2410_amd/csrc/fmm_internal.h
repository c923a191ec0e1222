// Internal declarations of the gfx950 FMM library: tree layout, workspace, and the
// kernel launchers implemented in kernels.hip.  Not part of the C ABI.
#pragma once

#include <hip/hip_runtime.h>

#include <array>
#include <atomic>
#include <functional>
#include <memory>
#include <cstdint>
#include <string>
#include <vector>

#include "device_cache.h"
#include "host_tree.h"
#include "morton.h"

namespace fmm {

constexpr int kMaxDepth = 12;
constexpr int kMaxP = 32;
constexpr int kNumEvents = 8;


// ---------------------------------------------------------------------------------
// Device-side tables for one expansion order p (radius-scaled operators, level
// independent):
//   M2M: A_m = sum_{k<=m} C(m,k) d_q^(m-k) 2^-k a_k
//   L2L: b_k = sum_{l>=k} C(l,k) d_q^(l-k) 2^-(k+1) b_l
//   M2L: b_l = sum_m (-1)^l C(l+m,m) delta^-(l+m+1) a_m,  delta = (dx, dy)
// with d_q = (c_child - c_parent)/w_parent = ((q&1) - 1/2)/2 + i((q>>1) - 1/2)/2, as
// 2p x 2p real matrices (complex entries embedded with interleaved (re, im) rows and
// columns, zero-padded) in the operand order of the matrix instructions
// (translate.hip), slots 0..48 the M2L offsets (index (dx+3)*7 + (dy+3)), 49..52 the L2L parities, 53..56
// the M2M children.
// ---------------------------------------------------------------------------------
struct Tables {
    int p = 0;
    float *mfma_f = nullptr;
    double *mfma_d = nullptr;
    int4 *mfma_entries = nullptr;  // {dx, dy, slot, kind}: 4 x 28 M2L/L2L entries, then 4 M2M entries
    double *zero_row = nullptr;    // 128 zero doubles: the row read for absent source cells
};

// Coefficient arrays are allocated with this many extra elements at the end, so that
// fixed-length reads of a row never pass the allocation.
constexpr int64_t kCoefPad = 64;
// The number of XCDs that workgroups are dealt to round-robin.
constexpr int kXcds = 8;
constexpr int64_t kLastLevelCacheBytes = int64_t(256) << 20;  // MI355X Infinity Cache

// Whether a call's per-particle outputs (bytes_per_row each) reach user order through the
// staging windows (written by sorted bucket, then gathered in user order) rather than by
// random rows: once they fill the last-level cache.  At 2^24 patch particles (16-byte
// velocities: exactly the cache) the windows measured faster, 8.44 -> 8.36 ms per
// evaluation, and the adjoint's 24 (40) bytes 18.30 -> 18.15 (23.85 -> 23.50) ms.
inline bool outputs_windowed(int64_t n, int64_t bytes_per_row)
{
    return n * bytes_per_row >= kLastLevelCacheBytes;
}
// Whether per-particle rows go between user and sorted order directly (random rows of an array that
// the caches hold) rather than through a staging pass of its own, whose launch costs 3 to 5 us: up
// to 8 MiB of rows, twice the L2 of an XCD.  Forward (circulations of 8 bytes): 4096 particles 48 ->
// 42 us, 500001 170 -> 155, 1000001 244 -> 232, 2000001 463 -> 459; adjoint (cotangents of 16):
// 500001 269 -> 265 us, 2^20 394 -> 408.
constexpr int64_t kDirectBytes = int64_t(8) << 20;
constexpr int64_t kForwardRow = 8, kAdjointRow = 16;
inline bool direct_rows(int64_t n, int64_t row) { return n * row <= kDirectBytes; }

// Where the circulation of sorted particle i is: rows[idx[i]], in the caller's array (idx = perm) or
// in the staging array (idx = gpos2).
struct GammaRows {
    const int *idx = nullptr;
    const double *rows = nullptr;
};
// Blocks of the reduction that finds the range of an adjoint's charges.
constexpr int kRangeBlocks = 1024;
// Flag (in w) of a mutual item in the near-field work list.
constexpr int kMutualItem = 256;

// A mutual item of leaves of many tiles is one wavefront's serial chain: 700001 patch particles
// in FP64, one tight patch: the heaviest item is 10816 steps and all items together 8000 per
// SIMD.  So items of more than twice kSplitShare-th of a SIMD's share of the near field's cost
// (and of more than kSplitLeast, four blocks of tiles) are cut into parts of about that
// cost, each a range of the tiles of the leaf with more of them (R) against all of S, an entry
// of its own.  A part's sums for R are whole and go to R's slot; those for S go to an array of
// the part's own and are added up by a kernel after the near field, in the order of the parts.
// Entry: kMutualItem | (1 + its place in the list) << 9.
constexpr int kSplitShare = 8, kSplitSimds = 1024;
constexpr int64_t kSplitLeast = 768;
struct MutualParts {
    const int4 *list = nullptr;  // {first and end particle of R, first place in sums, -}; NULL: none
    void *sums = nullptr;        // count pairs of sums, then count third sums
    int64_t count = 0;
};

// Owner value of a workspace handed to a tree over other particles (clear before use).
constexpr uint64_t kForeignOwner = ~uint64_t(0);

// Coefficient storage for one (p, precision, split) configuration.  Levels 0..split
// are FP64, levels split+1..L are FP32; each level holds 4^l cells x p coefficients,
// multipoles (scaled a_m / w^m) and locals (scaled b_l w^(l+1)) in separate arrays.
struct Workspace {
    int p = 0, precision = -1, split = -1;
    // serial number of the tree whose call last wrote the multipoles (0: none yet, or
    // unknown after a hand-over): another tree must clear them first, since each call
    // writes only the cells that are non-empty in its own tree
    uint64_t owner = 0;
    void *gam = nullptr;          // circulations in tree order in the near field's precision, n
    double2 *stage = nullptr;     // n: the velocities in tree order before the permutation to user order
    double2 *near = nullptr;      // near-field (u, v) per sorted particle, n
    double2 *mp_d = nullptr, *lo_d = nullptr;  // FP64 levels
    float2 *mp_f = nullptr, *lo_f = nullptr;   // FP32 levels
    // backward pass
    double2 *adj = nullptr;       // per sorted particle: adjoint charge q (sorted order)
    double4 *bwd_near = nullptr;  // per sorted particle: near sums of Im Phi, A (2) and B
    double2 *mp2_d = nullptr, *lo2_d = nullptr;  // the expansions of the charges q
    float2 *mp2_f = nullptr, *lo2_f = nullptr;
    void *rec2 = nullptr;         // adjoint charges q in FP32 for the mixed near field
    double4 *bwd_src = nullptr;   // per sorted particle: near sums of the source-position terms
    // One region for the per-particle sums of either call: the forward's mutual near-field
    // slots (9 x n float2 or double2) or the adjoint's near sums (bwd_near, bwd_src),
    // never live in the same call.
    void *sums = nullptr;
    size_t sums_bytes = 0;
    void *slots = nullptr;        // = sums
    void *phi_slots = nullptr;    // the pair force with Phi: 9 x n sums in the near field's precision
    double2 *range = nullptr;     // kRangeBlocks block maxima of |Gamma| and |q|, then their power of two
};

}  // namespace fmm

struct fmm_tree {
    int64_t n = 0;
    bool pooled = false;  // tree arrays from the stream-ordered pool (the device build)
    int depth = 0;
    double x0 = 0, y0 = 0, side = 1;
    int device = 0;
    int num_cus = 256;   // compute units of the device
    int lc = 3;          // coarse-level cutoff L_c
    int schedule = 2;    // 0 overlap, 1 serial, 2 by the cost model (FMM_OPT_SCHEDULE)
    int near_mutual = 1; // pairs of dense leaves evaluated once for both particles
    int dense_leaf = 32; // a leaf with at least this many particles is dense
    int near_occupancy = -1; // cap on forward near-field wavefronts per SIMD beside the far field
                             // (0: none, -1: chosen per call from the cost model)
    int occupancy_in_use = 0; // the cap of the current call (0 when serialised)
    int timing = 0;
    int validate = 0;    // FMM_OPT_VALIDATE: check circulations (and dL/du) for NaN / Inf first
    std::atomic<int> busy{0};
    // the tree's arrays were released by a rebuild that failed after the position checks:
    // only fmm_rebuild_tree and fmm_destroy_tree accept the handle
    bool released = false;

    // host statistics
    int64_t p2p_pairs = 0, m2l_pairs = 0, nonempty_leaves = 0, max_leaf = 0;
    int64_t nunits = 0;
    std::vector<int64_t> list_off;  // per level l: offset into d_lists; list_len[l] entries
    std::vector<int64_t> list_len;
    std::vector<int64_t> class_off; // per level l: 4 entries, start of each parity class inside the level list

    // device tree arrays; of the device build those of fixed size are parts of `slab`
    char *slab = nullptr;
    int64_t cap_lists = 0, cap_units = 0, cap_tile_box = 0, cap_near_work = 0;  // elements they have room for
    void *pos_buf[2] = {nullptr, nullptr};  // memory of d_pos
    int *d_perm = nullptr;        // sorted slot -> user index
    // Two-pass permutation of the circulations into sorted order through a staging array
    // cut into buckets of 2^stage_shift consecutive sorted slots (at most kStageBuckets):
    int stage_shift = 0;
    int *d_gpos1 = nullptr;       // user index -> staging slot (inside a bucket: by user index)
    int *d_gpos2 = nullptr;       // sorted slot -> staging slot of its user index
    double *d_st1 = nullptr;      // staging array, n FP64
    int *d_leaf_of = nullptr;     // sorted slot -> leaf Morton index
    double2 *d_xy = nullptr;      // sorted positions
    int *d_leaf_start = nullptr;  // CSR over Morton-ordered leaves, 4^L + 1
    int *d_counts = nullptr;      // particles per cell, all levels, global cell index
    int *d_lists = nullptr;       // non-empty cells per level (levels 2..L), parity-grouped
    int4 *d_units = nullptr;      // P2P work units {leaf, first, count, log2 lanes per target}
    // near-field plan of the mutual form (see build_near_plan)
    int64_t nunits_tc = 0, nmut = 0, nnear_work = 0;
    // split mutual items (MutualParts), the places in the parts' sums
    int64_t nsplit = 0, npart_sums = 0;
    int4 *d_split = nullptr, *d_parts = nullptr;
    double *d_part_sums = nullptr;  // 3 per place
    int64_t cap_split = 0, cap_parts = 0, cap_part_sums = 0;
    int64_t mutual_pairs = 0;     // ordered pairs (i != j) evaluated by the mutual items
    int4 *d_near_work = nullptr;  // mutual items and target-centric units, heaviest first
    uint16_t *d_leaf_mask = nullptr; // per leaf: bit d slot d written, bit 9 target-centric part
    int *d_tile_start = nullptr;  // per leaf: index of its first 64-particle tile, 4^L + 1
    float4 *d_tile_box = nullptr; // per tile: {xmin, ymin, xmax, ymax} in leaf units about the leaf centre
    int *d_flag = nullptr;        // result of the input check (FMM_OPT_VALIDATE)
    // leaf-unit coordinates xi = (z - c_leaf)/w_L of the sorted particles, float2 [0] and
    // double2 [1], each made on the first evaluation in that precision
    void *d_pos[2] = {nullptr, nullptr};

    fmm::SideStream aux;  // side stream and events, from the library's cache

    const fmm::Tables *tabs = nullptr;  // shared, never freed by the tree
    // evaluation workspace, shared by the trees of fmm_share_workspace (freed with the last)
    std::shared_ptr<fmm::Workspace> wsp = std::make_shared<fmm::Workspace>();
    uint64_t serial = 0;  // unique per tree of the process
    std::vector<std::array<hipEvent_t, fmm::kNumEvents>> pending_timing;
};

namespace fmm {

// Outputs of an adjoint call, in user order (device pointers, each may be null):
//   dg   dL/dGamma, added to the array when acc_g (else written);
//   dxe  dL/dx at the evaluation points, dxs dL/dx of the sources (written);
//   dxy  their sum, the derivative for particles moving as both, plus lam (when given: the
//        identity part of a transport stage x + h u(x)), added to the array when acc_xy.
// The cotangent is scaled before the sums, so every part but lam carries that scale.
struct AdjointOut {
    double *dg = nullptr, *dxe = nullptr, *dxs = nullptr, *dxy = nullptr;
    const double *lam = nullptr;
    int acc_g = 0, acc_xy = 0;
};

// The near field of the pair force (dl_dxy without its two parts): the target-centric part and
// the slots as the forward's (mask NULL: no slots), the same for the sums of Phi when dl_dgamma
// is asked for (phi not NULL), and the power of two the FP32 charges carry (NULL: none).
struct ForceNear {
    double2 *near = nullptr;
    const uint16_t *mask = nullptr;
    void *slots = nullptr;
    double *phi = nullptr;
    void *phi_slots = nullptr;
    const double *qscale = nullptr;
};

// Launch parameters shared by the forward and backward far-field chains.
struct FarArgs {
    const fmm_tree *t;
    int p;
    int split;                 // last FP64 level
    double2 *mp_d, *lo_d;      // FP64 storage (levels 0..split)
    float2 *mp_f, *lo_f;       // FP32 storage (levels split+1..L)
    const void *pos;           // the tree's leaf-unit coordinates in the records' precision (or null)
    const void *gam;           // circulations in tree order in that precision (null: P2M reads `gamma`)
    int rec_is_double;
    const double2 *adj;        // complex charges in sorted order (null: real circulations, c = -i Gamma/(2 pi))
    GammaRows gamma{};         // the circulations
    bool no_lds = false;       // beside a capped near field, which holds the LDS: kernels without any
};

// Launchers (kernels.hip).  All are asynchronous on `s`.
// Stages 1-3 on the device (tree_build.hip); the near-field plan from the device leaf
// offsets (used by both builds).  FMM_* status; err / bad_index describe a failure.
// after_checks (if set) runs once the positions have passed their checks (inside the
// root cell, finite), before the sorted arrays are made: a rebuild takes over the old
// tree's arrays there.
int build_tree_device(fmm_tree *t, const double *xy, const double *root_box, hipStream_t s, std::string &err,
                      int64_t &bad_index, const std::function<void()> &after_checks = {});
int build_near_plan_device(fmm_tree *t, hipStream_t s, std::string &err);

// Pass 1 of the circulations into tree order (the staging array, all P2M needs), then
// pass 2 with the near-field records.
// The circulations: staged unless direct_rows; then gathered into tree order.
GammaRows launch_stage_in(const fmm_tree *t, const double *gamma, int64_t row, hipStream_t s);
void launch_pack(const fmm_tree *t, const GammaRows &gamma, int is_double, void *gam, hipStream_t s);
// The tree's leaf-unit coordinates (float2 or double2, n) into pos.
void launch_leaf_coords(const fmm_tree *t, int is_double, void *pos, hipStream_t s);
void launch_p2p_forward(const fmm_tree *t, const void *pos, const void *gam, int is_double, double alpha,
                        double2 *near, void *slots, hipStream_t s);
// Stages 4-7 (P2M, M2M, M2L, L2L).
// b: a second set of expansions (its own storage and charges, the rest as a's), in the same launches.
void launch_far_chain(const FarArgs &a, hipStream_t s, const FarArgs *b = nullptr);
// uv alone is written through `stage` (a buffer of n double2); with base, uv = base + h u.
void launch_finalize(const fmm_tree *t, const FarArgs &a, const double2 *near, const void *slots, int slots_double,
                     double alpha, double *uv, double *uv_near, double *uv_far, void *stage, const double *base,
                     double h, hipStream_t s);

// Backward
// The two passes between user and sorted order through bucket staging windows (gpos1,
// gpos2 and the shift of a sorted order): rows of one or two doubles from user order into
// their staging slots, and staged double2 rows out to user order (uv = base + h row with
// base, else the row).
void launch_stage_rows(int64_t n, int shift, const int *gpos1, const double *src, double *st, hipStream_t s);
void launch_stage_rows2(int64_t n, int shift, const int *gpos1, const double2 *src, double2 *st, hipStream_t s);
void launch_gather_rows(int64_t n, const int *gpos1, const double2 *staged, double *uv, const double *base, double h,
                        hipStream_t s);
void launch_adjoint_range(int64_t n, const double *gamma, const double *dl_duv, double scale, double2 *range,
                          hipStream_t s);
void launch_pack_adjoint(const fmm_tree *t, const double *dl_duv, double scale, double2 *adj, void *qt, int is_double,
                         double2 *staging, const double2 *range, double *qscale, hipStream_t s);
void launch_p2p_force(const fmm_tree *t, const void *pos, const void *gam, const void *qv, const double2 *adj,
                      const GammaRows &gamma, int is_double, double alpha, const ForceNear &near, hipStream_t s);
void launch_finalize_force(const fmm_tree *t, const FarArgs &fc, const FarArgs &fq, const double2 *adj,
                           const ForceNear &near, int is_double, double alpha, const AdjointOut &out, hipStream_t s);
void launch_p2p_backward(const fmm_tree *t, const void *pos, const void *gam, const void *qv, int is_double,
                         double alpha, double4 *out_pa, double4 *out_src, hipStream_t s);
void launch_finalize_backward(const fmm_tree *t, const FarArgs &fc, const FarArgs &fq, const double4 *near_pa,
                              const double2 *adj, const double4 *near_src, int is_double,
                              double alpha, const AdjointOut &out, double *stage_g, double *stage_x,
                              double *stage_s, hipStream_t s);

// Lowest index k of the n groups of `stride` doubles at a (device) that holds a NaN or an
// infinity, or -1 in bad; flag is a device int of the caller.  Synchronises s.
hipError_t find_nonfinite(const double *a, int64_t n, int stride, int *flag, hipStream_t s, int64_t &bad);

// Tables (host generation + upload), kernels.hip
int upload_tables(Tables &tb, int p, std::string &err);
void free_tables(Tables &tb);
// The tables of p-term expansions on a device (the current one): built on first use, shared
// by every tree of the process and kept until it ends.  Returns 0, -2 (no memory) or -3;
// with create false, -5 when they do not exist yet (nothing is allocated).
int shared_tables(int device, int p, const Tables **out, std::string &err, bool create = true);

// The library's static device workspace (fmm_velocity_noalloc): its address on the
// current device (looked up once per device) and its size in bytes.  hipError_t status.
constexpr size_t kStaticWorkspaceBytes = size_t(128) << 20;
int static_workspace(int device, char **base);
// Zero `bytes` (a multiple of 8) at p with a kernel (no memset node, no allocation).
void launch_zero(void *p, size_t bytes, hipStream_t s);

}  // namespace fmm
