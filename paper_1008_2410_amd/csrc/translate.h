// Translations of the expansions (stages 5-7: M2M, M2L, L2L) on the matrix cores, shared by
// the uniform and the adaptive tree.  Launchers in translate.hip.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "fmm_internal.h"

namespace fmm {

// One class of one level's target list: targets[start .. start + len), in tiles from tile0
// on.  Classes of a level are in parity order, so segment index & 3 is the parity of its
// targets in the M2L and L2L launches.
struct TransSeg {
    int tile0, start, len, level;
};

// One launch over up to kMaxTransSegs segments (4 parity classes of every level).
constexpr int kMaxTransSegs = 4 * 17;

struct TransArgs {
    int nseg = 0, ntiles = 0, p = 0;
    bool no_lds = false;              // launch no kernel that uses LDS (a capped near field holds it)
    const int *targets = nullptr;     // target cells (uniform tree: Morton index within the level)
    const int4 *entries = nullptr;    // {dx, dy, slot, kind}
    const void *tab = nullptr;        // operators in MFMA operand order, FP64 or FP32
    const double *zero = nullptr;     // the row of absent sources
    const void *src = nullptr;        // source rows (M2L, M2M: multipoles; L2L: the parents' locals)
    void *out = nullptr;              // target rows
    int64_t src_off = 0, out_off = 0; // uniform tree: global cell index of row 0 of src / out
    const void *par = nullptr;        // uniform tree, M2L of one level: the parents' locals, for its L2L as well
    int64_t par_off = 0;
    // the same for a second set of expansions, in the same launch (the adjoint's two chains)
    const void *src2 = nullptr, *par2 = nullptr;
    void *out2 = nullptr;
    // adaptive tree
    const int *vslot = nullptr;       // 27 source cells per cell of level >= 2 (cell - first)
    const int *x_off = nullptr;       // cells with an X list start from their P2L sums
    const int *parent = nullptr;
    const int4 *child = nullptr;
    int first = 0;
    TransSeg seg[kMaxTransSegs];
};

// Three levels of the upward or downward pass, a workgroup per cell of level `base` and its
// descendants.
struct SubtreeArgs {
    int p, base, deepest;             // deepest: last level read (up) or written (down)
    const int *counts;                // uniform tree: occupancy by global cell index
    double *rows;                     // FP64 rows from cell 0: multipoles (up) or locals (down)
    double *rows2 = nullptr;          // a second set of them, in the same launch
    const double *tab;
    // adaptive tree
    const int *cells = nullptr;       // the split cells of level `base`
    int ncells = 0;
    const int4 *child = nullptr;
    const double *zero = nullptr;     // the row of absent cells
};

// Tables of p terms: KS(p) steps of four rows and columns in blocks of 16 (FP64), KF(p)
// steps of two rows and columns in blocks of 32 (FP32).
inline int trans_ks(int p) { return p <= 8 ? 4 : p <= 12 ? 6 : p <= 16 ? 8 : p <= 24 ? 12 : 16; }
inline int trans_kf(int p) { return p <= 8 ? 8 : p <= 12 ? 12 : p <= 16 ? 16 : p <= 24 ? 24 : 32; }
inline int trans_cols64(int p) { return (4 * trans_ks(p) + 15) / 16 * 16; }
inline int trans_cols32(int p) { return p <= 16 ? 32 : 64; }

enum class Trans { M2L, M2M, L2L };

// Whether a level of `cells` targets fills the chip by itself (1024 SIMDs twice over): its
// M2L and L2L are then one launch, which saves writing and reading its locals once; below,
// the M2L of all such levels is one launch and the L2L follows level by level.
inline bool wide_level64(int64_t cells, int p) { return cells / 16 * (trans_cols64(p) / 16) >= 2048; }
inline bool wide_level32(int64_t cells, int p) { return cells / 32 * (trans_cols32(p) / 32) >= 2048; }

// FP64 launches (tiles of 16 targets, or 32 in a wide M2L: see launch_trans64), adaptive:
// the source cells come from vslot / child / parent instead of the cell's position.
void launch_trans64(TransArgs a, Trans mode, bool adaptive, hipStream_t s);
// FP32 products (tiles of 32 targets) of the uniform tree: M2L on FP32 rows; M2M from FP32
// children into FP32 or FP64 parents (out_double); L2L from FP32 or FP64 parents
// (src_double) into FP32 children.  An M2L with `par` (rows of its own precision) takes the
// L2L along.
void launch_trans32(TransArgs a, Trans mode, bool src_double, bool out_double, hipStream_t s);
// Levels base + 2 .. base of the upward pass, or base + 1 .. base + 3 of the downward pass
// (at most to `deepest`), a workgroup per cell of level `base` (adaptive tree: per split cell).
void launch_subtree(const SubtreeArgs &a, bool up, hipStream_t s);

}  // namespace fmm
